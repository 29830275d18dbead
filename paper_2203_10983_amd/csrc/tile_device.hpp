// Device code of a layer's forward pass on a tile of a few rows: see tile.hip.
#pragma once
#include "spmm_device.hpp"
#include "split_bf16.hpp"

namespace bns {

constexpr int kTileRows = 16, kTileWaves = 8;
constexpr int kTileDepth = 128;  // widest input row
constexpr int kTileLd = kTileDepth + 4;  // 4 floats on from row to row: the 64 operands of an instruction are in 64 banks

struct TileArgs {
  SpmmArgs sp;
  const float *W;       // [d_in, d_out]; SAGE: [2 d_in, d_out], neighbour half first
  const float *H_self;  // SAGE: the layer's input
  float *H_out;
  int32_t d_out, rows;  // rows of a tile
  bool relu;
  bool concat;          // SAGE: both halves of the update are one chain of sums (else two, added)
  Dropout drop;
  TileLoss loss;
};

// The gradient of one node's cross-entropy from its logits z, by LPR lanes that hold up to four classes each: the steps and the order of
// sums of softmax_ce_kernel.  Returns the node's loss on lane 0 of the group.
template <int LPR>
__device__ __forceinline__ float ce_row(const float *z, int C, int y, bool ok, float *g, float *gp, int ld) {
  const int sl = lane_id() % LPR;
  float x[4], m = -INFINITY, se = 0.f, zy = 0.f;  // y: negative outside the training set
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = sl + k * LPR;
    x[k] = ok && c < C ? z[c] : -INFINITY;
    m = fmaxf(m, x[k]);
  }
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, kWave));
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = sl + k * LPR;
    if (c == y) zy = x[k];
    x[k] = c < C ? expf(x[k] - m) : 0.f;
    se += x[k];
  }
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) {
    se += __shfl_xor(se, off, kWave);
    zy += __shfl_xor(zy, off, kWave);
  }
  if (!ok) return 0.f;
  const float inv = 1.f / se;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = sl + k * LPR;
    const float o = y < 0 || c >= C ? 0.f : x[k] * inv - (c == y ? 1.f : 0.f);
    if (c < C) g[c] = o;
    if (gp && c < ld) gp[c] = o;
  }
  return sl == 0 && y >= 0 ? (m + logf(se)) - zy : 0.f;
}

// Lanes per node, and the node of a tile that a lane has a share of: one pass takes a whole tile.
__device__ __forceinline__ int ce_lanes(int C) { return C <= 32 ? 8 : C <= 64 ? 16 : 32; }
__device__ __forceinline__ int ce_node(int C) { return threadIdx.x / ce_lanes(C); }
static_assert(kTileWaves * kWave / 32 >= kTileRows && kTileLossWidth <= 4 * 32);

typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

// The rows row0 .. + rows of the aggregate, in the order of sums of spmm_kernel: put(row, piece, sums) on the lanes that hold
// them.  Rows from a.n_split on are kept boundary rows of a transposed aggregate.
template <int LPR, typename Put>
__device__ __forceinline__ void gather_tile(const SpmmArgs &a, int row0, int rows, Put put) {
  using V = typename Vec<4>::T;
  const int lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane / LPR, sl = lane % LPR;
  const int d = a.d, nvec = d / 4;
  auto entries = [&](int row, int &e0, int &e1) {
    const int2 ee = scalar_load_pair(a.row_ptr, row);
    const InnerWeights iw = inner_weights(a, row, ee.x, ee.y);
    e0 = ee.x;
    e1 = ee.y;
    if (a.row_skip) e0 += scalar_load(a.row_skip, row);
    if (a.row_take) e1 = e0 + scalar_load(a.row_take, row);
    return iw;
  };
  float acc[1][4];
  if (a.plan.n_multi == 0 || row0 >= a.n_split) {
    for (int r = wid; r < rows; r += kTileWaves) {
      int e0, e1;
      const InnerWeights iw = entries(row0 + r, e0, e1);
      gather_segment<4, 1, LPR>(a, row0 + r, iw, e0, e1, 0, nvec, acc);
      if (g == 0) put(row0 + r, sl, acc);
    }
    return;
  }
  // a wavefront per segment; the sums of rows of several segments are added in ascending order
  const int end = scalar_load(a.plan.seg_ptr, row0 + rows);
  for (int u = scalar_load(a.plan.seg_ptr, row0) + wid; u < end; u += kTileWaves) {
    const int2 unit = scalar_load(a.plan.seg_unit, u);
    const int row = unit.x, slot = unit.y;
    int e0, e1;
    const InnerWeights iw = entries(row, e0, e1);
    if (slot >= 0) {
      const int seg = slot - scalar_load(a.plan.part_ptr, row);
      const int2 ss = scalar_load_pair(a.plan.seg_ptr, row);
      const int chunk = (e1 - e0 + (ss.y - ss.x) - 1) / (ss.y - ss.x);
      e0 = min(e1, e0 + seg * chunk);
      e1 = min(e1, e0 + chunk);
    }
    gather_segment<4, 1, LPR>(a, row, iw, e0, e1, 0, nvec, acc);
    if (g != 0) continue;
    if (slot < 0) put(row, sl, acc);
    else if (sl < nvec) reinterpret_cast<V *>(a.partials + (size_t)slot * d)[sl] = V{acc[0][0], acc[0][1], acc[0][2], acc[0][3]};
  }
  __syncthreads();
  for (int r = wid; r < rows; r += kTileWaves) {
    const int row = row0 + r;
    const int2 ss = scalar_load_pair(a.plan.seg_ptr, row);
    const int nseg = ss.y - ss.x;
    if (nseg <= 1) continue;
    const float *part = a.partials + (size_t)scalar_load(a.plan.part_ptr, row) * d;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[0][i] = 0.f;
    if (lane < nvec)
      for (int s = 0; s < nseg; ++s) {
        const V x = reinterpret_cast<const V *>(part + (size_t)s * d)[lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[0][i] += x[i];
      }
    put(row, lane, acc);
  }
}

// A layer's forward pass on one tile.  LOSS: also the softmax cross-entropy of the last layer's output and its gradient.  tile_no, thread: the tile's number and
// that of a thread among its kTileWaves wavefronts; As: its rows.  gather(row0, rows, put): gather_tile or what takes its place.  Every thread of the workgroup gets to the same barriers, also where a tile has no rows.
template <int LPR, int VW, bool SAGE, bool LOSS, typename Gather>
__device__ __forceinline__ void tile_layer(const TileArgs &f, int tile_no, int thread, float (&As)[SAGE ? 2 : 1][kTileRows * kTileLd], Gather gather) {
  using V = typename Vec<4>::T;
  const SpmmArgs &a = f.sp;
  const int lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(thread >> 6);
  const int d = a.d, nvec = d / 4, N = f.d_out;
  const int row0 = tile_no * f.rows, rows = min(f.rows, a.n_split - row0);

  // ---- the wavefront's columns of W: a lane holds VW of them at depths 4 m + lane / 16 ----
  const int l16 = lane & 15, g4 = lane >> 4;
  const int n0 = wid * 16 * VW;
  const int col = min(n0 + l16 * VW, N - VW);  // lanes past the last column repeat it
  float w[LPR][VW];  // d / 4 <= LPR
  auto load_w = [&](const float *Wm) {
    if (n0 >= N) return;
    const float *p = Wm + (size_t)g4 * N + col;
#pragma unroll
    for (int m = 0; m < LPR; ++m)
      if (m < nvec) {
        if constexpr (VW == 2) {
          const f32x2u x = *reinterpret_cast<const f32x2u *>(p + (size_t)(4 * m) * N);
          w[m][0] = x[0];
          w[m][1] = x[1];
        } else {
          w[m][0] = p[(size_t)(4 * m) * N];
        }
      }
  };
  load_w(f.W);
  int label = -1;
  if constexpr (LOSS)
    if (ce_node(N) < rows) label = f.loss.labels[row0 + ce_node(N)];
  if constexpr (SAGE) {  // the rows' own features
    for (int idx = thread; idx < rows * nvec; idx += kTileWaves * kWave) {
      const int r = idx / nvec, c4 = idx - r * nvec;
      *reinterpret_cast<V *>(&As[1][r * kTileLd + c4 * 4]) = reinterpret_cast<const V *>(f.H_self + (size_t)(row0 + r) * d)[c4];
    }
  }

  gather(row0, rows, [&](int row, int piece, const float (&acc)[1][4]) {  // as finish_row, and into the tile
    const float scale = a.out_scale0 ? scalar_load(a.out_scale0, row) : 1.f;
    if (piece >= nvec) return;
    V o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = acc[0][i];
    if (a.init) o += reinterpret_cast<const V *>(a.init + (size_t)row * d)[piece];
    o *= scale;
    *reinterpret_cast<V *>(&As[0][(row - row0) * kTileLd + piece * 4]) = o;
    reinterpret_cast<V *>(a.out0 + (size_t)row * d)[piece] = o;
  });
  __syncthreads();
  if (!LOSS && n0 >= N) return;

  // ---- update ----
  f32x4 sum[VW];
#pragma unroll
  for (int c = 0; c < VW; ++c) sum[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto product = [&](const float *tile) {
    if (LOSS && n0 >= N) return;
    // (the tile's rows past the last one hold anything: an operand's row is one result's row)
    const float *as = tile + l16 * kTileLd + g4;
#pragma unroll
    for (int m = 0; m < LPR; ++m)
      if (m < nvec) {
        const float x = as[4 * m];
#pragma unroll
        for (int c = 0; c < VW; ++c) sum[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, w[m][c], sum[c], 0, 0, 0);
      }
  };
  product(As[0]);
  if constexpr (SAGE) {
    load_w(f.W + (size_t)d * N);
    f32x4 first[VW];
#pragma unroll
    for (int c = 0; c < VW; ++c) {
      first[c] = f.concat ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[c];
      if (!f.concat) sum[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    product(As[1]);
    if (!f.concat)
#pragma unroll
      for (int c = 0; c < VW; ++c) sum[c] += first[c];
  }
  // a lane holds rows 4 (lane / 16) .. + 3 of its columns
  __shared__ float Zs[LOSS ? kTileRows * kTileLd : 1];
  float loss = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int lrow = 4 * g4 + r;
    float x[VW];
#pragma unroll
    for (int c = 0; c < VW; ++c) {
      x[c] = sum[c][r];
      if (f.relu) {
        x[c] = fmaxf(x[c], 0.f);
        if (f.drop.scale != 0.f) x[c] = dropout_keeps(f.drop, row0 + lrow, col + c) ? x[c] * f.drop.scale : 0.f;
      }
    }
    if (lrow >= rows || (LOSS && n0 + l16 >= N)) continue;
    float *const to = f.H_out + (size_t)(row0 + lrow) * N + col;
    if constexpr (VW == 2) *reinterpret_cast<f32x2u *>(to) = f32x2u{x[0], x[1]};
    else *to = x[0];
    if constexpr (LOSS) Zs[lrow * kTileLd + col] = x[0];
  }
  if constexpr (LOSS) {
    __syncthreads();
    const TileLoss &l = f.loss;
    const int node = ce_node(N);
    const bool ok = node < rows;
    const float *z = Zs + (ok ? node : 0) * kTileLd;
    const size_t row = row0 + (ok ? node : 0);
    float *const g = l.dZ + row * N, *const gp = l.dZ_pad ? l.dZ_pad + row * l.ld : nullptr;
    if (N <= 32) loss = ce_row<8>(z, N, label, ok, g, gp, l.ld);
    else if (N <= 64) loss = ce_row<16>(z, N, label, ok, g, gp, l.ld);
    else loss = ce_row<32>(z, N, label, ok, g, gp, l.ld);
    loss = wave_sum(loss);
    __shared__ float part[kTileWaves];
    if (lane == 0) part[wid] = loss;
    __syncthreads();
    if (threadIdx.x == 0) {
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < kTileWaves; ++i) sum += part[i];
      f.loss.partials[tile_no] = sum;
    }
  }
}

// Half a tile where whole ones are fewer than the compute units: a row per wavefront (steps of 128-128-128-47, forward layers in tiles of
// 16 and 8, us: 1000 rows 66 / 64, of 45 entries 93 / 84; 3000 92 / 91; 4500 98 / 106).
inline int tile_rows(int32_t n) { return n <= 3584 ? kTileRows / 2 : kTileRows; }

}  // namespace bns
