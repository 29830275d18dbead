// Loss summed over the inner nodes (Algorithm 1, loss step) with its gradient, the ReLU mask of
// the backward pass and the Adam update.  The loss is reduced in a
// fixed order (per wavefront, per block, then one block over the block partials): two runs give
// the same bits.
#include <algorithm>
#include <cmath>

#include "device_utils.hpp"
#include "kernels.hpp"
#include "pack_device.hpp"

namespace bns {

constexpr int kT = 256;

__device__ __forceinline__ float block_sum_fixed(float x) {  // valid on thread 0
  __shared__ float part[kT / kWave];
  x = wave_sum(x);
  if (lane_id() == 0) part[threadIdx.x / kWave] = x;
  __syncthreads();
  float s = 0.f;
  if (threadIdx.x == 0)
#pragma unroll
    for (int w = 0; w < kT / kWave; ++w) s += part[w];
  __syncthreads();
  return s;
}

// softmax cross-entropy: loss_v = logsumexp(z_v) - z_v[y_v], dZ_v = softmax(z_v) - onehot(y_v).
// LPR lanes per node hold its row in registers, up to four classes each (C <= 4 LPR): one read, one write, bound by
// memory.  With a whole wavefront per node whatever the width, 306 250 rows of 47 classes took 74 us and their padded copy another
// 28 (pad_rows); together now 40.
template <int LPR>
__global__ void __launch_bounds__(kT)
softmax_ce_kernel(int n, int C, const float *__restrict__ logits, const int32_t *__restrict__ labels,
                  float *__restrict__ dZ, int ld, float *__restrict__ dZ_pad, float *__restrict__ partials) {
  constexpr int R = 2;  // rows of a lane group per step, their loads and reductions interleaved
  const int sl = threadIdx.x % LPR;
  const int groups = gridDim.x * (kT / LPR);
  auto group_sum = [](float x) {
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
    return x;
  };
  auto group_max = [](float x) {
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, kWave));
    return x;
  };
  float loss_acc = 0.f;  // meaningful on lane 0 of the group
  for (int v = blockIdx.x * (kT / LPR) + threadIdx.x / LPR; v < n; v += R * groups) {
    int row[R], y[R];
    float x[R][4], m[R], se[R], zy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      row[r] = v + r * groups;
      const bool ok = row[r] < n;
      y[r] = ok ? labels[row[r]] : -1;
      m[r] = -INFINITY;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = sl + k * LPR;
        x[r][k] = (ok && c < C) ? logits[(size_t)row[r] * C + c] : -INFINITY;
        m[r] = fmaxf(m[r], x[r][k]);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) m[r] = group_max(m[r]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      se[r] = 0.f;
      zy[r] = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = sl + k * LPR;
        if (c == y[r]) zy[r] = x[r][k];
        x[r][k] = c < C ? expf(x[r][k] - m[r]) : 0.f;
        se[r] += x[r][k];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      se[r] = group_sum(se[r]);
      zy[r] = group_sum(zy[r]);  // exactly one lane holds z[y]; the others add zeros
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (row[r] >= n) continue;
      float *g = dZ + (size_t)row[r] * C;
      float *gp = dZ_pad + (size_t)row[r] * ld;
      const float inv = 1.f / se[r];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = sl + k * LPR;
        // a node outside the training set (negative label): no loss, zero gradient
        const float o = y[r] < 0 || c >= C ? 0.f : x[r][k] * inv - (c == y[r] ? 1.f : 0.f);
        if (c < C) g[c] = o;
        if (dZ_pad && c < ld) gp[c] = o;
      }
      if (sl == 0 && y[r] >= 0) loss_acc += (m[r] + logf(se[r])) - zy[r];
    }
  }
  const float s = block_sum_fixed(sl == 0 ? loss_acc : 0.f);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// More than 256 classes: a wavefront per node, the row read three times.
__global__ void __launch_bounds__(kT)
softmax_ce_wide_kernel(int n, int C, const float *__restrict__ logits, const int32_t *__restrict__ labels,
                       float *__restrict__ dZ, float *__restrict__ partials) {
  const int lane = lane_id();
  const int waves = gridDim.x * (kT / kWave);
  float loss_acc = 0.f;  // meaningful on lane 0
  for (int v = blockIdx.x * (kT / kWave) + threadIdx.x / kWave; v < n; v += waves) {
    const float *z = logits + (size_t)v * C;
    float *g = dZ + (size_t)v * C;
    const int y = labels[v];
    if (y < 0) {  // node outside the training set: no loss, zero gradient
      for (int c = lane; c < C; c += kWave) g[c] = 0.f;
      continue;
    }
    float m = -INFINITY;
    for (int c = lane; c < C; c += kWave) m = fmaxf(m, z[c]);
    m = wave_max(m);
    float se = 0.f;
    for (int c = lane; c < C; c += kWave) se += expf(z[c] - m);
    se = wave_sum(se);
    const float inv = 1.f / se;
    for (int c = lane; c < C; c += kWave) g[c] = expf(z[c] - m) * inv - (c == y ? 1.f : 0.f);
    if (lane == 0) loss_acc += (m + logf(se)) - z[y];
  }
  const float s = block_sum_fixed(lane == 0 ? loss_acc : 0.f);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// sigmoid binary cross-entropy over nodes x labels:
// loss = max(z,0) - z*y + log(1 + exp(-|z|)),  dZ = sigmoid(z) - y
__global__ void __launch_bounds__(kT)
sigmoid_bce_kernel(int64_t total, const float *__restrict__ logits, const uint8_t *__restrict__ labels,
                   float *__restrict__ dZ, int C, int ld, float *__restrict__ dZ_pad, float *__restrict__ partials) {
  const int64_t stride = (int64_t)gridDim.x * kT;
  float acc = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < total; i += stride) {
    const float z = logits[i];
    float g = 0.f;
    if (labels[i] != 255) {  // 255: entry outside the training set
      const float y = (float)labels[i];
      const float e = expf(-fabsf(z));
      acc += fmaxf(z, 0.f) - z * y + log1pf(e);
      const float sig = z >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
      g = sig - y;
    }
    dZ[i] = g;
    if (dZ_pad) {
      const int64_t row = i / C;
      const int c = (int)(i - row * C);
      float *gp = dZ_pad + row * ld;
      gp[c] = g;
      if (c == C - 1)
        for (int k = C; k < ld; ++k) gp[k] = 0.f;
    }
  }
  const float s = block_sum_fixed(acc);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

hipError_t loss_softmax_ce(int32_t n, int32_t C, const float *logits, const int32_t *labels,
                           float *dZ, int32_t ld, float *dZ_pad, float *partials, int32_t *n_partials, hipStream_t s) {
  if (dZ_pad && (ld < C || ld > (C + 3) / 4 * 4 || C > 256)) return hipErrorInvalidValue;
  // two nodes per lane group at a time; no more workgroups than there is work for
  const int lpr = C <= 32 ? 8 : C <= 64 ? 16 : C <= 128 ? 32 : 64;
  const int64_t per_block = 2 * (kT / lpr);
  const int64_t blocks = std::min<int64_t>(kLossBlocks, ((int64_t)n + per_block - 1) / per_block);
#define BNS_CE(LPR) softmax_ce_kernel<LPR><<<(unsigned)blocks, kT, 0, s>>>(n, C, logits, labels, dZ, ld, dZ_pad, partials)
  if (C > 256) softmax_ce_wide_kernel<<<(unsigned)blocks, kT, 0, s>>>(n, C, logits, labels, dZ, partials);
  else if (lpr == 8) BNS_CE(8);
  else if (lpr == 16) BNS_CE(16);
  else if (lpr == 32) BNS_CE(32);
  else BNS_CE(64);
#undef BNS_CE
  *n_partials = (int32_t)blocks;
  return hipGetLastError();
}

hipError_t loss_sigmoid_bce(int32_t n, int32_t C, const float *logits, const uint8_t *labels,
                            float *dZ, int32_t ld, float *dZ_pad, float *partials, int32_t *n_partials, hipStream_t s) {
  if (dZ_pad && ld < C) return hipErrorInvalidValue;
  const int64_t total = (int64_t)n * C, blocks = std::min<int64_t>(kLossBlocks, (total + kT - 1) / kT);
  sigmoid_bce_kernel<<<(unsigned)blocks, kT, 0, s>>>(total, logits, labels, dZ, C, ld, dZ_pad, partials);
  *n_partials = (int32_t)blocks;
  return hipGetLastError();
}

// one thread and one draw per element
__global__ void __launch_bounds__(kT)
dropout_inplace_kernel(int n_rows, int d, float *__restrict__ H, const Dropout drop) {
  const int64_t total = (int64_t)n_rows * d;
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const int row = (int)(i / d), col = (int)(i - (int64_t)row * d);
  const float x = H[i];
  H[i] = dropout_keeps(drop, row, col) ? x * drop.scale : 0.f;
}

hipError_t dropout_inplace(int32_t n_rows, int32_t d, float *H, const Dropout &drop, hipStream_t s) {
  if (drop.scale == 0.f || n_rows <= 0) return hipSuccess;
  const int64_t total = (int64_t)n_rows * d;
  dropout_inplace_kernel<<<(unsigned)((total + kT - 1) / kT), kT, 0, s>>>(n_rows, d, H, drop);
  return hipGetLastError();
}

// Four columns of a row per thread and turn, the gradient once more in padded rows on the way, which were a launch of 5 us (all
// calls of an iteration, with the count of the kept boundary entries beside the sampling: 20011 rows 602-130-66-9 582 -> 570 us,
// 477 rows 100-256-41 113 -> 106).  Rows without padding are one long row.
__global__ void __launch_bounds__(kT)
relu_mask_kernel(int64_t n_rows, int64_t d, int ld, const float *__restrict__ dH, const float *__restrict__ H, float scale,
                 float *__restrict__ out, float *__restrict__ pad, int blocks, const PackJobs pack) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  if ((int)blockIdx.x >= blocks) {
    pack_unit(pack, (blockIdx.x - blocks) * (kT / kWave) + threadIdx.x / kWave);
    return;
  }
  const int64_t pieces = pad ? ld / 4 : (d + 3) / 4, total = n_rows * pieces, stride = (int64_t)blocks * kT;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < total; i += stride) {
    const int64_t r = pad ? i / pieces : 0, c = (i - r * pieces) * 4, at = r * d + c;
    f4 g = {0.f, 0.f, 0.f, 0.f};
    if (c + 4 <= d) {
      g = *reinterpret_cast<const f4u *>(dH + at);
      if (H) {
        const f4 h = *reinterpret_cast<const f4u *>(H + at);
#pragma unroll
        for (int e = 0; e < 4; ++e) g[e] = h[e] > 0.f ? g[e] * scale : 0.f;
        *reinterpret_cast<f4u *>(out + at) = g;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (c + e < d) {
          g[e] = dH[at + e];
          if (H) out[at + e] = g[e] = H[at + e] > 0.f ? g[e] * scale : 0.f;
        }
    }
    if (pad) *reinterpret_cast<f4 *>(pad + r * ld + c) = g;
  }
}

hipError_t relu_mask(int32_t n_rows, int32_t d, const float *dH, const float *H, float scale, float *out, int32_t ld, float *pad,
                     const PackJobs &pack, hipStream_t s) {
  if (n_rows <= 0) return hipSuccess;
  if (pad && (ld < d || ld % 4 != 0)) return hipErrorInvalidValue;
  const int64_t rows = pad ? n_rows : 1, row = pad ? d : (int64_t)n_rows * d, pieces = rows * (pad ? ld / 4 : (row + 3) / 4);
  const int64_t blocks = H || pad ? std::min<int64_t>((pieces + kT - 1) / kT, 65536) : 0;
  const unsigned grid = (unsigned)(blocks + (pack.units + kT / kWave - 1) / (kT / kWave));
  if (grid) relu_mask_kernel<<<grid, kT, 0, s>>>(rows, row, ld, dH, H, scale, out, pad, (int)blocks, pack);
  return hipGetLastError();
}

// Adam (Kingma & Ba, 2015): m <- b1 m + (1-b1) g, v <- b2 v + (1-b2) g^2,
// w <- w - lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps)
__global__ void __launch_bounds__(kT)
adam_kernel(int64_t n, float *__restrict__ W, const float *__restrict__ dW, float *__restrict__ m,
            float *__restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  const float g = dW[i];
  const float mi = b1 * m[i] + (1.f - b1) * g;
  const float vi = b2 * v[i] + (1.f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  W[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

__global__ void __launch_bounds__(kT)
sgd_kernel(int64_t n, float *__restrict__ W, const float *__restrict__ dW, float lr) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < n) W[i] -= lr * dW[i];
}
hipError_t sgd_update(int64_t n, float *W, const float *dW, float lr, hipStream_t s) {
  if (n > 0) sgd_kernel<<<(unsigned)((n + kT - 1) / kT), kT, 0, s>>>(n, W, dW, lr);
  return hipGetLastError();
}

hipError_t adam_update(int64_t n, float *W, const float *dW, float *m, float *v, float lr, float b1,
                       float b2, float eps, int32_t t, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const float c1 = (float)(1.0 / (1.0 - pow((double)b1, (double)t)));
  const float c2 = (float)(1.0 / (1.0 - pow((double)b2, (double)t)));
  adam_kernel<<<(unsigned)((n + kT - 1) / kT), kT, 0, s>>>(n, W, dW, m, v, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

__global__ void counter_kernel(uint32_t *counter, uint32_t value) { *counter = value; }
hipError_t set_counter(uint32_t *counter, uint32_t value, hipStream_t s) {
  counter_kernel<<<1, 1, 0, s>>>(counter, value);
  return hipGetLastError();
}

}  // namespace bns
