// The backward products of the update (Eq. 2), and the forward one of the last layer, on the matrix cores: fp32 operands and
// results, products by three-way bf16 splitting (split_bf16.hpp).
//
//   gemm_rows   C = A B   dA = dZ W^T, H = [A | A2] W: a tall A [M, K] times a weight matrix, which
//               pack_weights has split and laid out as operand fragments
//   gemm_tn     C = [A | A2]^T B  weight gradient dW = A^T dZ, the depth (rows) split over the chip
//
// gemm_rows: a workgroup of 4 wavefronts walks row tiles; a wavefront owns 16 R rows and NC column
// tiles of 16.  Its rows come straight from global memory into the operand layout (a lane reads two
// 16-byte pieces of its row per 32-deep step, four lanes of a row 64 contiguous bytes) and are split in
// registers, each element once.  The packed weights of a step go from L2 straight into a
// double-buffered LDS tile shared by the four wavefronts, one step ahead, across row tiles as well; those of a product of a
// single step (K <= 32) are copied once and stay, without a wait or a barrier per tile.
// The weight fragment is the first operand of the instruction, so a lane ends up with four
// consecutive columns of one row; lanes of neighbouring rows trade pieces so that whole lines are stored (pieces of 64 bytes:
// 578125 rows of 128 columns at depth 128 146 us, lines 128; at depth 16 65 and 58).
//
// gemm_tn: a thread reads 16-byte pieces of eight consecutive-depth rows of one operand, which makes
// it hold eight depths of four columns: after the split each column's eight values are one 16-byte
// fragment entry in LDS.  The partial tiles are stored as the accumulators lie in the registers;
// one kernel adds them in a fixed order and puts the elements where they belong.
//
// What bounds them: the 128-wide products move 1 KB per row for 32 k flops and are bound by memory (dZ W^T on 578125 rows
// 117 us, 5.1 TB/s; A^T dZ 128), the 512-wide ones by the matrix cores, six bf16 instructions per fp32 product (at the
// dense rate 417 TFLOP/s of fp32 products): 89625 x 512 x 512 205 us (229 TFLOP/s) and 236 (199), where the splitting
// beside the instructions takes the rest.
//
// Both ask for a step's rows while the one before is multiplied, and that only holds while no read stands behind a branch of
// its own: where the last columns and rows, and rows by index, had such branches, the reads were waited for one by one.  Without
// them, us: A^T dZ of 197758 rows by index x 602 x 256 547 -> 400, 306250 x 128 x 47 99 -> 62, 128 x 128 145 -> 117, 578125 x 128 x 172
// 213 -> 170, 9570 rows of three layers 20 -> 15; dZ W^T of 578125 x 172 x 128 190 -> 173, 306250 x 47 x 128 102 -> 94.
// It takes registers: the 128 x 128 tiles of A^T dZ and the forward products of 32 rows by 128 columns have three on the stack, which they
// did not before (89625 x 512 x 512 265 -> 236 all the same).
#include <algorithm>
#include <type_traits>

#include "device_utils.hpp"
#include "kernels.hpp"
#include "pack_device.hpp"
#include "split_bf16.hpp"

namespace bns {

// ---- packed weights -----------------------------------------------------------------------------
size_t packed_bytes(int32_t K, int32_t N) { return (size_t)k_steps(K) * col_tiles(N) * kFragSet; }
size_t packed_bytes_f32(int32_t K, int32_t N) { return (size_t)k_steps(K) * ((N + 31) / 32) * 4096; }

__global__ void __launch_bounds__(256) pack_weights_kernel(const PackJobs jobs) {
  pack_unit(jobs, blockIdx.x * 4 + (threadIdx.x >> 6));
}

hipError_t pack_weights(const PackJobs &jobs, hipStream_t s) {
  if (jobs.units) pack_weights_kernel<<<(unsigned)((jobs.units + 3) / 4), 256, 0, s>>>(jobs);
  return hipGetLastError();
}

// ---- rows x packed weights ------------------------------------------------------------------------
struct RowsArgs {
  RowsGemm g;
  int T, S, nblk;  // column tiles, depth steps, column blocks
};

// kTwo: the depth of C's rows goes on in A2 (below).  The last three are a forward product's: with ReLU and dropout, added to what is there, with a
// second set of rows by record.
enum RowsEpilogue { kPlain, kMask, kPair, kTwo, kFwd, kFwdAdd, kFwdRec };

// The value of the lane whose number differs in the last bit.
__device__ __forceinline__ float quad_swap(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xb1, 0xf, 0xf, true));  // quad_perm:[1,0,3,2]
}

// Adds ReLU and dropout and stores `left` (0 to 4) of the columns col .. col + 3 of a row of a forward product.  All lanes draw for the dropout, those that
// store nothing too: a wavefront with few of its lanes active takes longer over it.
template <bool ADD>
__device__ __forceinline__ void fwd_store(const RowsGemm &p, f32x4 v, int left, int row, int col, float *d) {
  if constexpr (ADD) {
    if (left == 4) v += *reinterpret_cast<const f32x4u *>(d);
    else
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (e < left) v[e] += d[e];
  }
  if (p.relu) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
    if (p.drop.scale != 0.f) {
#pragma unroll 1
      for (int e = 0; e < 4; ++e) {
        const float y = dropout_keeps(p.drop, row, col + e) ? v[0] * p.drop.scale : 0.f;
        v = f32x4{v[1], v[2], v[3], y};
      }
    }
  }
  if (left == 4) *reinterpret_cast<f32x4u *>(d) = v;
  else
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (e < left) d[e] = v[e];
}

template <int R, int NC, int EPI>
__global__ void __launch_bounds__(256, R * NC > 8 || NC > 6 ? 3 : 4) gemm_rows_kernel(const RowsArgs a) {
  constexpr int kRows = 64 * R;  // rows of a workgroup's tile
  __shared__ __attribute__((aligned(16))) char Bs[2][NC * kFragSet];
  const RowsGemm &p = a.g;
  constexpr bool kForward = EPI >= kFwd, kMore = EPI != kPair && EPI != kFwd && EPI != kFwdAdd;
  const int M = p.M, M2 = kMore && p.A_more ? min(p.M2, *p.m2_dev) : 0;
  // workgroup b runs on XCD b % 8: the column blocks of one row tile follow each other on one XCD, so
  // that they find its rows in that XCD's L2
  const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
  const int nb = q % a.nblk, stride = (gridDim.x / (8 * a.nblk)) * 8;
  const int t0 = nb * NC;
  int tile = (q / a.nblk) * 8 + x;
  const int n_first = (M + kRows - 1) / kRows;  // row tiles of C; those of C_more follow
  const int n_tiles = n_first + (M2 + kRows - 1) / kRows;
  if (tile >= n_tiles) return;

  const int lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  // kTwo: a row of C takes the steps of A, then those of A2; a row of C_more those of A_more alone
  auto steps_of = [&](int tl) { return EPI == kTwo && tl < n_first ? 2 * a.S : a.S; };
  int S = steps_of(tile);

  f32x4 ar[R][2];
  const float *row_a[R], *row_a2[R];
  float row_scale[R];  // kFwdRec: of the rows whose values ar holds
  const bool two = kForward && p.A2 != nullptr;  // then a_split % 16 == 0
  auto set_rows = [&](int tl) {
    const bool more = kMore && tl >= n_first;
    const float *A = more ? p.A_more : p.A;
    const int end = more ? M2 : M, first = (more ? tl - n_first : tl) * kRows;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      int row = min(end - 1, first + wid * 16 * R + r * 16 + l16);  // rows past the end are not stored
      row_scale[r] = 1.f;
      if (EPI == kFwdRec && more) {
        const int2 rec = p.rec[row];
        row = rec.x;
        row_scale[r] = __int_as_float(rec.y);
      }
      row_a[r] = A + (size_t)row * p.lda;
      if (EPI == kFwd) row_a2[r] = two ? p.A2 + (size_t)row * p.lda - p.a_split : nullptr;
      if (EPI == kTwo) row_a2[r] = more ? row_a[r] : p.A2 + (size_t)row * p.lda;
    }
  };
  auto step_in = [&](int s) { return EPI == kTwo && s >= a.S ? s - a.S : s; };  // of its operand
  auto load_a = [&](int step) {
    const int s = step_in(step);
    const float *from[R];
#pragma unroll
    for (int r = 0; r < R; ++r) from[r] = EPI == kTwo && step >= a.S ? row_a2[r] : row_a[r];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int k = s * 32 + j * 16 + g * 4;
      if ((s + 1) * 32 <= p.K) {
#pragma unroll
        for (int r = 0; r < R; ++r) ar[r][j] = *reinterpret_cast<const f32x4u *>((EPI == kFwd && two && s * 32 + j * 16 >= p.a_split ? row_a2[r] : from[r]) + k);
      } else if (p.K >= 4) {  // settle() takes what is past the end away
#pragma unroll
        for (int r = 0; r < R; ++r) ar[r][j] = *reinterpret_cast<const f32x4u *>(from[r] + piece_start(k, p.K));
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int e = 0; e < 4; ++e) ar[r][j][e] = k + e < p.K ? from[r][k + e] : 0.f;
      }
    }
  };
  auto settle = [&](int step) {
    const int s = step_in(step);
    if constexpr (EPI == kFwdRec)
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < 2; ++j) ar[r][j] *= row_scale[r];
    if ((s + 1) * 32 <= p.K || p.K < 4) return;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < R; ++r) ar[r][j] = row_end(ar[r][j], s * 32 + j * 16 + g * 4, p.K);
  };
  const unsigned lds0 = lds_offset_of(&Bs[0][0]);
  const int nt = min(NC, a.T - t0);  // column tiles of this block (uniform)
  auto load_b = [&](int s, int buf) {  // pieces of 1 KB, dealt to the four wavefronts
    const char *src = static_cast<const char *>(p.Bp) + (size_t)(s * a.T + t0) * kFragSet + lane * 16;
    for (int c = wid; c < nt * 3; c += 4)
      lds_dma16(src + c * kFragBytes, lds0 + buf * (NC * kFragSet) + c * kFragBytes);
  };

  f32x4 acc[NC][R];
  auto clear = [&]() {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < R; ++r) acc[c][r] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  const bool stay = EPI != kTwo && a.S == 1;  // the weights of a single step stay in LDS for all tiles
  set_rows(tile);
  load_b(0, 0);
  load_a(0);
  clear();
  if (stay) {
    lds_dma_wait();
    __syncthreads();
  }
  int buf = 0;
  for (int s = 0;;) {
    Frag3 fa[R];
    if (!stay) {
      lds_dma_wait();
      __syncthreads();  // this step's weights are in LDS, and everybody is done with the other buffer
    }
    settle(s);
#pragma unroll
    for (int r = 0; r < R; ++r) fa[r] = split8(ar[r][0], ar[r][1]);
    const bool last = s + 1 == S;
    const int ntile = last ? tile + stride : tile, ns = last ? 0 : s + 1;
    if (ntile < n_tiles) {
      if (last) set_rows(ntile);
      if (!stay) load_b(ns, buf ^ 1);
      load_a(ns);
    }
    const char *bs = &Bs[buf][0] + lane * 16;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Frag3 fb;
#pragma unroll
      for (int i = 0; i < 3; ++i) fb.p[i] = *reinterpret_cast<const bf16x8 *>(bs + c * kFragSet + i * kFragBytes);
      f32x4 part[R];
      mfma_split<R>(part, fb, fa);
#pragma unroll
      for (int r = 0; r < R; ++r) acc[c][r] += part[r];
    }
    buf = stay ? ns : buf ^ 1;
    if (last) {
      // A lane holds columns 16 c + 4 g .. + 3 of row l16 for every tile c.  Of two tiles it trades one with the lane of the
      // row beside its own, so that eight lanes hold 128 consecutive bytes of one row.
      constexpr bool kTrade = NC > 1;
      constexpr int W = kTrade ? 2 : 1, NP = (NC + W - 1) / W;  // tiles, and rows, of a trade
      const int odd = kTrade ? l16 & 1 : 0;
      const int n_end = EPI == kFwdRec && p.pad ? p.ldc : p.N, col0 = (t0 + odd) * 16 + g * 4;  // pad: the packed weights are zero there
      const bool more = kMore && tile >= n_first;
      const int end = more ? M2 : M, row0 = (more ? tile - n_first : tile) * kRows + wid * 16 * R + l16 - odd;
      const float scale = more ? 1.f : p.alpha;
      const float alpha = (t0 + odd) & 1 ? -scale : scale;  // odd tiles are summed negated
      float nonfinite = 0.f;
      unsigned again = 0;  // forward: pieces to be formed once more, which are not stored before
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < NP; ++c) {
          f32x4 out[W];
          if constexpr (kTrade) {
            const f32x4 x = acc[2 * c][r], y = 2 * c + 1 < NC ? acc[2 * c + 1 < NC ? 2 * c + 1 : 0][r] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float got = quad_swap(odd ? x[e] : y[e]);
              out[0][e] = odd ? got : x[e];
              out[W - 1][e] = odd ? y[e] : got;
            }
          } else {
            out[0] = acc[c][r];
          }
          const int col = col0 + c * 16 * W;
          const int left = c * W + odd < nt ? n_end - col : 0;  // columns from this lane's first one to the end; none of other blocks' tiles
#pragma unroll
          for (int h = 0; h < W; ++h) {
            const int row = row0 + r * 16 + h;
            f32x4 v = out[h];
            const size_t at = (size_t)row * p.ldc + col;
            const float a = W == 1 && (t0 + c) & 1 ? -scale : alpha;
            if constexpr (kForward) {
              float *const d = (more ? p.C_more : p.C) + at;
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] *= a;
              const bool in = row < end && left > 0;
              if (in && (nonfinite_seed(0.f, v) != 0.f || any_tiny(v))) {
                again |= 1u << ((r * NP + c) * W + h);
                continue;
              }
              fwd_store<EPI == kFwdAdd>(p, v, in ? min(left, 4) : 0, row, col, d);
              continue;
            }
            if (row >= end || left <= 0) continue;
            nonfinite = nonfinite_seed(nonfinite, v);
            if ((EPI == kMask || (EPI == kTwo && p.mask)) && !more) {
              const float *const ms = p.mask + at;
              f32x4 m = {0.f, 0.f, 0.f, 0.f};
              if (left >= 4) m = *reinterpret_cast<const f32x4u *>(ms);
              else
#pragma unroll
                for (int e = 0; e < 3; ++e)
                  if (e < left) m[e] = ms[e];
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = m[e] > 0.f ? v[e] * a : 0.f;
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] *= a;
            }
            float *const d = (EPI == kPair && col >= p.c_split ? p.C2 - p.c_split : more ? p.C_more : p.C) + at;  // c_split % 4 == 0
            if (left >= 4) *reinterpret_cast<f32x4u *>(d) = v;
            else
#pragma unroll
              for (int e = 0; e < 3; ++e)
                if (e < left) d[e] = v[e];
          }
        }
      if constexpr (kForward) {
#pragma unroll 1
        for (; again; again &= again - 1) {
          const int q = __ffs(again) - 1, c = q / W % NP, row = row0 + q / (NP * W) * 16 + q % W, col = col0 + c * 16 * W;
          const int left = min(4, n_end - col);
          int row_in = row;
          const float *A = more ? p.A_more : p.A;
          float by = 1.f;
          if (EPI == kFwdRec && more) {
            const int2 rec = p.rec[row];
            row_in = rec.x;
            by = __int_as_float(rec.y);
          }
          f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
          for (int k = 0; k < p.K; ++k) {
            const float *const from = two && k >= p.a_split ? p.A2 - p.a_split : A;
            const float y = from[(size_t)row_in * p.lda + k] * by;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = col + e < p.N ? fmaf(y, p.W[(size_t)k * p.N + col + e], x[e]) : 0.f;
          }
          fwd_store<EPI == kFwdAdd>(p, x, left, row, col, (more ? p.C_more : p.C) + (size_t)row * p.ldc + col);
        }
      } else if (nonfinite != 0.f) {  // (NaN)
        const float *A = more ? p.A_more : p.A;
#pragma unroll 1
        for (int q = 0; q < R * NP * W; ++q) {
          const int c = q / W % NP, row = row0 + q / (NP * W) * 16 + q % W, col = col0 + c * 16 * W;
          const int left = c * W + odd < nt ? n_end - col : 0;
          if (row >= end || left <= 0) continue;
          float *const d = (EPI == kPair && col >= p.c_split ? p.C2 - p.c_split : more ? p.C_more : p.C) + (size_t)row * p.ldc + col;
          bool fine = true;
#pragma unroll
          for (int e = 0; e < 4; ++e) fine &= e >= left || is_finite(d[e]);
          if (fine) continue;
          const float *const w = p.W + (size_t)col * p.K;
          float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
          for (int k = 0; k < p.K; ++k) {
            const float y = A[(size_t)row * p.K + k];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = fmaf(y, w[(e < left ? (size_t)e * p.K : 0) + k], x[e]);
          }
          if (EPI == kTwo && !more) {
            const float *const w2 = w + (size_t)p.N * p.K;
#pragma unroll 1
            for (int k = 0; k < p.K; ++k) {
              const float y = p.A2[(size_t)row * p.K + k];
#pragma unroll
              for (int e = 0; e < 4; ++e) x[e] = fmaf(y, w2[(e < left ? (size_t)e * p.K : 0) + k], x[e]);
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (e < left && !is_finite(d[e])) d[e] = x[e] * scale;
        }
      }
      if (ntile >= n_tiles) break;
      clear();
      tile = ntile;
      S = steps_of(tile);
    }
    s = ns;
  }
}

template <int R, int EPI>
static void launch_rows(const RowsArgs &a, int nc, unsigned grid, hipStream_t s) {
  switch (nc) {
    case 1: gemm_rows_kernel<R, 1, EPI><<<grid, 256, 0, s>>>(a); break;
    case 2: gemm_rows_kernel<R, 2, EPI><<<grid, 256, 0, s>>>(a); break;
    case 3: gemm_rows_kernel<R, 3, EPI><<<grid, 256, 0, s>>>(a); break;
    case 4: gemm_rows_kernel<R, 4, EPI><<<grid, 256, 0, s>>>(a); break;
    case 5: gemm_rows_kernel<R, 5, EPI><<<grid, 256, 0, s>>>(a); break;
    case 6: gemm_rows_kernel<R, 6, EPI><<<grid, 256, 0, s>>>(a); break;
    case 7: gemm_rows_kernel<R, 7, EPI><<<grid, 256, 0, s>>>(a); break;
    default: gemm_rows_kernel<R, 8, EPI><<<grid, 256, 0, s>>>(a); break;
  }
}
template <int R>
static void launch_rows(const RowsArgs &a, int nc, unsigned grid, hipStream_t s) {
  if (a.g.fwd && (a.g.rec || a.g.pad)) launch_rows<R, kFwdRec>(a, nc, grid, s);
  else if (a.g.fwd && a.g.accumulate) launch_rows<R, kFwdAdd>(a, nc, grid, s);
  else if (a.g.fwd) launch_rows<R, kFwd>(a, nc, grid, s);
  else if (a.g.C2) launch_rows<R, kPair>(a, nc, grid, s);
  else if (a.g.A2) launch_rows<R, kTwo>(a, nc, grid, s);
  else if (a.g.mask) launch_rows<R, kMask>(a, nc, grid, s);
  else launch_rows<R, kPlain>(a, nc, grid, s);
}

hipError_t gemm_rows(const RowsGemm &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.C2 ? g.c_split % 4 != 0 || g.ldc < g.c_split || g.N > 2 * g.c_split : g.ldc < g.N) return hipErrorInvalidValue;
  if (g.C2 && (g.mask || g.A_more)) return hipErrorInvalidValue;
  if (g.fwd ? g.C2 || g.mask || g.lda < (g.A2 ? g.a_split : g.K) || (g.A2 && (g.a_split % 16 != 0 || g.K != 2 * g.a_split)) ||
                  (g.A2 && (g.accumulate || g.rec)) || (g.rec && (g.accumulate || g.relu || !g.m2_dev)) || (g.A_more && !g.rec) ||
                  (g.pad && (g.ldc > (g.N + 3) / 4 * 4 || g.A2 || g.relu || g.accumulate))
            : (g.A2 && g.C2) || g.rec || g.relu || g.pad || g.accumulate || g.lda != g.K)
    return hipErrorInvalidValue;
  RowsArgs a;
  a.g = g;
  a.T = col_tiles(g.N);
  a.S = k_steps(g.K);
  // Up to 8 column tiles per wavefront, evenly dealt.  Where that leaves the chip short of workgroups
  // (three fit a compute unit), smaller tiles: first half the rows, then half the columns.
  constexpr int kWanted = 512;
  a.nblk = (a.T + 7) / 8;
  int R = 2;
  const int64_t m2 = g.A_more ? g.m2_expected : 0;
  auto row_tiles = [&]() { return (g.M + 64 * R - 1) / (64 * R) + (m2 + 64 * R - 1) / (64 * R); };
  auto groups = [&]() { return row_tiles() * a.nblk; };
  if (groups() < kWanted) R = 1;
  while (groups() < kWanted && a.nblk * 2 <= a.T) a.nblk *= 2;
  int nc = (a.T + a.nblk - 1) / a.nblk;
  a.nblk = (a.T + nc - 1) / nc;
  // A grid of whole octets of row tiles, every column block of each; the tiles past one resident round are walked.  A
  // single step in a single column block is over before the next tile's rows have come: a workgroup per tile there
  // (128 columns at depth 16: 578125 rows 65 -> 58 us; 512 columns, four blocks, 89625 rows: 42 us, 38 when walked).
  int64_t octets = (row_tiles() + 7) / 8;
  if (a.S > 1 || a.nblk > 1) octets = std::min<int64_t>(octets, std::max<int64_t>(1, 768 / (8 * a.nblk)));
  const unsigned grid = (unsigned)(octets * 8 * a.nblk);
  if (R == 2) launch_rows<2>(a, nc, grid, s);
  else launch_rows<1>(a, nc, grid, s);
  return hipGetLastError();
}

hipError_t gemm_fwd_split(const RowsF32 &f, const float *W, hipStream_t s) {
  RowsGemm g{};
  g.fwd = true;
  g.M = f.M; g.N = f.N; g.K = f.K; g.A = f.A; g.W = W; g.Bp = f.Bp; g.C = f.C; g.ldc = f.ldc;
  g.alpha = 1.f;
  g.A2 = f.A2; g.a_split = f.a_split; g.lda = f.lda;
  g.relu = f.relu; g.pad = f.pad; g.accumulate = f.accumulate; g.drop = f.drop;
  g.rec = f.rec; g.A_more = f.A_rec; g.C_more = f.C_rec; g.M2 = f.M2; g.m2_expected = f.m2_expected; g.m2_dev = f.m2_dev;
  return gemm_rows(g, s);
}

// ---- transposed products, depth split over the chip ----------------------------------------------
// The weight gradients of a training step are independent of each other and of the backward chain once
// its gradients are known, so all of them run as one batch: one launch of the products per tile shape (the
// splits dealt by work), one launch that adds up every partial.
struct TnJob {
  const float *A, *A2, *B;
  const int32_t *rows, *k_dev;
  float *partials;
  int M, N, K, a_split, lda;
  int tiles_n, nt, splits;
  int first;  // first workgroup of the job
};
struct TnJobs {
  TnJob j[kMaxTnJobs];
  int n;
};

// Bytes between the fragment sets of neighbouring 16-column tiles in LDS: 64 more than a set, so
// that the eight lanes that store together (four columns of two tiles) hit different banks.
constexpr int kTnTile = kFragSet + 64;

template <int MB, int NB>
__global__ void __launch_bounds__(256, 3) gemm_tn_kernel(const TnJobs jobs) {
  constexpr int KS = MB + NB > 128 ? 32 : 64;          // depth of a step: keeps all 256 threads loading
  constexpr int TM = MB / 16, TN = NB / 16, TILES = TM + TN;
  constexpr int GA = MB / 4, GB = NB / 4;              // 4-column groups of the two operands
  constexpr int KG = KS / 8;                           // groups of eight depths
  constexpr int MT = TM / 2, NT = TN / 2;              // 16 x 16 tiles of a wavefront (2 x 2 wavefronts)
  static_assert((GA + GB) * KG <= 256, "one load unit per thread");
  __shared__ __attribute__((aligned(16))) char lds[(KS / 32) * TILES * kTnTile];

  int q = 0;
  while (q + 1 < jobs.n && (int)blockIdx.x >= jobs.j[q + 1].first) ++q;
  const TnJob &a = jobs.j[q];
  const int b = (int)blockIdx.x - a.first;
  // the tiles of one depth chunk follow each other on one XCD (workgroup b runs on XCD b % 8)
  const int tile = (b >> 3) % a.nt, split = ((b >> 3) / a.nt) * 8 + (b & 7);
  if (split >= a.splits) return;
  const int m0 = (tile / a.tiles_n) * MB, n0 = (tile % a.tiles_n) * NB;
  const int K = a.k_dev ? min(a.K, *a.k_dev) : a.K;
  const int chunk = ((K + a.splits - 1) / a.splits + KS - 1) / KS * KS;  // from the real depth, which may live on the device
  const int k_begin = split * chunk, k_end = min(K, k_begin + chunk);

  // load unit of this thread: operand, 4-column group, group of eight depths
  const int t = threadIdx.x;
  const bool is_b = t >= GA * KG;
  const int u = is_b ? t - GA * KG : t;
  const int gcount = is_b ? GB : GA;
  const int c4 = u % gcount, kg = u / gcount;
  const bool active = kg < KG;
  const float *src;
  int ld, cols, width;  // columns in range at src (0..4), of the whole row
  if (is_b) {
    src = a.B + n0 + c4 * 4;
    ld = width = a.N;
    cols = a.N - (n0 + c4 * 4);
  } else {
    const int c = m0 + c4 * 4;
    src = a.A + c;
    ld = a.lda;
    width = a.A2 ? a.a_split : a.M;
    cols = width - c;
    if (a.A2 && cols <= 0) {
      src = a.A2 + c - a.a_split;
      cols = a.M - c;
    }
  }
  const bool straddle = !is_b && a.A2 && cols > 0 && cols < 4;  // a_split % 4 != 0: one group takes from both
  const int row_of_a2 = straddle ? m0 + c4 * 4 - a.a_split : 0;
  cols = straddle ? min(4, a.M - (m0 + c4 * 4)) : max(0, min(4, cols));
  const bool by_piece = !straddle && width >= 4;  // four columns at once, the last four of a row where fewer are left
  if (by_piece) src -= 4 - cols;
  // A's rows by index: the indices of two steps in LDS, asked for one step before the rows that wait for them
  __shared__ __attribute__((aligned(16))) int index[2][KS];
  const bool by_index = a.rows && !is_b;
  int next_index = 0;
  auto ask_index = [&](int k0) { return a.rows[min(k0 + t, k_end - 1)]; };
  const bool reads = active && cols > 0;
  f32x4 v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // (no branch around a single load: the next one would wait for it.  Rows past the end repeat the last one, settle() clears them)
  auto load = [&](int k0, int buf) {
    if (!reads) return;
    int r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = by_index ? index[buf][kg * 8 + j] : min(k0 + kg * 8 + j, k_end - 1);
    if (by_piece) {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const f32x4u *>(src + (size_t)r[j] * ld);
    } else {
      const float *at[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) at[e] = straddle && row_of_a2 + e >= 0 ? a.A2 + row_of_a2 + min(e, cols - 1) : src + min(e, cols - 1);
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][e] = at[e][(size_t)r[j] * ld];
    }
  };
  auto settle = [&](int k0) {
    const int k = k0 + kg * 8;
    if (!reads || (cols == 4 && k + 8 <= k_end)) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      f32x4 x = v[j];
      if (by_piece) x = row_end(x, 4 - cols, 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[j][e] = e < cols && k + j < k_end ? x[e] : 0.f;
    }
  };
  // column 4 c4 + i sits in slot 4 i + c4 % 4 of its tile (so that four lanes store 64 contiguous bytes)
  char *dst = lds + ((size_t)(kg / 4) * TILES + (is_b ? TM : 0) + c4 / 4) * kTnTile + ((kg & 3) * 16 + (c4 & 3)) * 16;
  // odd splits work on the negated A (mfma_split) and negate their sums when they store them
  auto stage = [&](auto neg) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const Frag3 f = split8<decltype(neg)::value>(f32x4{v[0][i], v[1][i], v[2][i], v[3][i]}, f32x4{v[4][i], v[5][i], v[6][i], v[7][i]});
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<bf16x8 *>(dst + p * kFragBytes + i * 64) = f.p[p];
    }
  };
  const bool neg = (split & 1) && !is_b;

  const int lane = lane_id(), wid = t >> 6, wm = wid >> 1, wn = wid & 1;
  f32x4 acc[NT][MT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (k_begin < k_end) {
    if (a.rows) {
      if (t < KS) {
        index[0][t] = ask_index(k_begin);
        index[1][t] = ask_index(k_begin + KS);
      }
      __syncthreads();
    }
    load(k_begin, 0);
  }
  int buf = 0;
  for (int k0 = k_begin; k0 < k_end; k0 += KS) {
    settle(k0);
    __syncthreads();  // the previous step's fragments have been read
    if (a.rows && t < KS && k0 > k_begin) index[buf ^ 1][t] = next_index;
    if (active) {
      if (neg) stage(std::true_type{});
      else stage(std::false_type{});
    }
    __syncthreads();
    buf ^= 1;
    if (k0 + KS < k_end) load(k0 + KS, buf);
    if (a.rows && t < KS) next_index = ask_index(k0 + 2 * KS);
#pragma unroll
    for (int ks = 0; ks < KS / 32; ++ks) {
      const char *base = lds + (size_t)ks * TILES * kTnTile + lane * 16;
      // A's tiles two at a time where the wavefront has more than eight results: the step's own sums beside the running
      // ones are 168 registers and 29 spilled with all four (A^T dZ of 89625 x 512 x 512: 273 us, 265 like this)
      constexpr int H = MT * NT > 8 ? 2 : MT;
#pragma unroll
      for (int h = 0; h < MT; h += H) {
        Frag3 fm[H];
#pragma unroll
        for (int i = 0; i < H; ++i)
#pragma unroll
          for (int p = 0; p < 3; ++p)
            fm[i].p[p] = *reinterpret_cast<const bf16x8 *>(base + (wm * MT + h + i) * kTnTile + p * kFragBytes);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          Frag3 fn;
#pragma unroll
          for (int p = 0; p < 3; ++p)
            fn.p[p] = *reinterpret_cast<const bf16x8 *>(base + (TM + wn * NT + j) * kTnTile + p * kFragBytes);
          f32x4 part[H];
          mfma_split<H>(part, fn, fm);
#pragma unroll
          for (int i = 0; i < H; ++i) acc[j][h + i] += part[i];
        }
        if (H < MT) asm volatile("" ::: "memory");  // B's fragments again
      }
    }
  }
  float *out = a.partials + (size_t)(split * a.nt + tile) * (MB * NB) + (size_t)wid * (MT * NT * 256) + lane * 4;
  float nonfinite = 0.f;
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      nonfinite = nonfinite_seed(nonfinite, acc[j][i]);
      *reinterpret_cast<f32x4 *>(out + (j * MT + i) * 256) = split & 1 ? -acc[j][i] : acc[j][i];
    }
  if (nonfinite != 0.f) {  // (NaN)
#pragma unroll 1
    for (int q = 0; q < NT * MT; ++q) {  // the elements of tile (j, i) as gemm_tn_reduce_kernel places them
      const int j = q / MT, i = q % MT, sa = lane & 15;
      const int m = m0 + (wm * MT + i) * 16 + 4 * (sa & 3) + (sa >> 2), n = n0 + (wn * NT + j) * 16 + (lane >> 4);  // n + 4 e
      if (m >= a.M || n >= a.N) continue;
      float *const d = out + q * 256;
      if (is_finite(d[0]) && is_finite(d[1]) && is_finite(d[2]) && is_finite(d[3])) continue;
      const float *A = a.A2 && m >= a.a_split ? a.A2 + (m - a.a_split) : a.A + m;
      float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
      for (int k = k_begin; k < k_end; ++k) {
        const float y = A[(size_t)(a.rows ? a.rows[k] : k) * a.lda];
        const float *const b = a.B + (size_t)k * a.N + n;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = fmaf(y, b[n + 4 * e < a.N ? 4 * e : 0], x[e]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!is_finite(d[e])) d[e] = x[e];
    }
  }
}

// The sums over the splits, in a fixed order: C = sum (+ the sum of the next job, for a gradient of two parts),
// optionally W -= lr * C (the plain update of Algorithm 1 takes its gradient from the registers).  A workgroup owns
// one 16 x 16 accumulator tile: NW wavefronts add every NW-th partial of it, then their sums are added
// in pairs.  One more workgroup adds up the partial losses of the step.
struct TnSum {
  const float *partials, *partials2;  // partials2 (nullable): the second part's, same tiles
  float *C, *W;
  int M, N, mt, nt_wave, tiles_n, nt, splits, splits2;  // mt x nt_wave accumulator tiles per wavefront
  int first;
};
struct TnSums {
  TnSum j[kMaxTnJobs];
  int n, blocks;
  float lr;
  TnLoss loss;
};

// The sum of the partial losses, by NW wavefronts; part: room for one float per wavefront.
template <int NW>
__device__ __forceinline__ void sum_loss(const TnLoss &loss, float *part) {
  const int lane = lane_id(), wid = threadIdx.x >> 6;
  float x = 0.f;
  for (int i = threadIdx.x; i < loss.n; i += NW * 64) x += loss.partials[i];
  x = wave_sum(x);
  if (lane == 0) part[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    float s = 0.f;
    for (int w = 0; w < NW; ++w) s += part[w];
    *loss.out = s;
    if (loss.bump) *loss.bump += 1;
  }
}

// a + b, c + d, ... in pairs, then the pairs.
template <int NW>
__device__ __forceinline__ float sum_in_pairs(const float (&part)[NW][256], int e) {
  float p[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) p[w] = part[w][e];
#pragma unroll
  for (int h = NW / 2; h > 0; h /= 2)
#pragma unroll
    for (int w = 0; w < h; ++w) p[w] += p[w + h];
  return p[0];
}

template <int NW>
__global__ void __launch_bounds__(NW * 64) gemm_tn_reduce_kernel(const TnSums jobs) {
  __shared__ float part[NW][256];
  const int lane = lane_id(), wid = threadIdx.x >> 6;
  if ((int)blockIdx.x == jobs.blocks) {
    sum_loss<NW>(jobs.loss, part[0]);
    return;
  }
  int q = 0;
  while (q + 1 < jobs.n && (int)blockIdx.x >= jobs.j[q + 1].first) ++q;
  const TnSum &a = jobs.j[q];
  const int F = 4 * a.mt * a.nt_wave;
  const int tile = ((int)blockIdx.x - a.first) / F, f = ((int)blockIdx.x - a.first) % F;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  auto add = [&](const float *partials, int splits) {
    const size_t stride = (size_t)a.nt * F * 256;
    const float *in = partials + ((size_t)tile * F + f) * 256 + lane * 4;
    constexpr int U = 4;
    for (int z0 = wid; z0 < splits; z0 += U * NW) {
      f32x4 x[U];
#pragma unroll
      for (int i = 0; i < U; ++i)
        x[i] = z0 + i * NW < splits ? *reinterpret_cast<const f32x4 *>(in + (size_t)(z0 + i * NW) * stride) : f32x4{0.f, 0.f, 0.f, 0.f};
      sum += (x[0] + x[1]) + (x[2] + x[3]);
    }
  };
  add(a.partials, a.splits);
  if (a.partials2) add(a.partials2, a.splits2);
  *reinterpret_cast<f32x4 *>(&part[wid][lane * 4]) = sum;
  __syncthreads();
  const int e = threadIdx.x;
  if (e >= 256) return;
  const float s = sum_in_pairs<NW>(part, e);
  // element e: lane e / 4, register e % 4; its slots in the two 16-column tiles are 4 (lane / 16) + e % 4
  // (columns of B) and lane % 16 (columns of A), slot q standing for column 4 (q % 4) + q / 4
  const int per_wave = a.mt * a.nt_wave, l = e >> 2, w4 = f / per_wave, ji = f % per_wave;
  const int j = ji / a.mt, i = ji % a.mt, sa = l & 15;
  const int m = (tile / a.tiles_n) * (32 * a.mt) + ((w4 >> 1) * a.mt + i) * 16 + 4 * (sa & 3) + (sa >> 2);
  const int n = (tile % a.tiles_n) * (32 * a.nt_wave) + ((w4 & 1) * a.nt_wave + j) * 16 + 4 * (e & 3) + (l >> 4);
  if (m >= a.M || n >= a.N) return;
  const size_t at = (size_t)m * a.N + n;
  a.C[at] = s;
  if (a.W) a.W[at] -= jobs.lr * s;
}

// ---- few rows: product and sum in one launch -------------------------------------------------------
// A workgroup of 16 wavefronts owns a tile of 16 x 16 of a gradient; wavefront w takes the depths 32 w .. + 31 of every 512 straight
// from memory into the operand layout (a lane reads eight depths of one column, 16 lanes 64 contiguous bytes of a row).
struct TnSmallJob {
  const float *A, *A2, *B;
  float *C, *W;
  int M, N, K, a_split, lda, tiles_n, first;
};
struct TnSmallJobs {
  TnSmallJob j[kMaxTnJobs];
  int n, blocks;
  float lr;
  TnLoss loss;
};
constexpr int kTnSmallWaves = 16;

__global__ void __launch_bounds__(kTnSmallWaves * kWave) gemm_tn_small_kernel(const TnSmallJobs jobs) {
  constexpr int NW = kTnSmallWaves;
  __shared__ float part[NW][256];
  const int lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x == jobs.blocks) {
    sum_loss<NW>(jobs.loss, part[0]);
    return;
  }
  int q = 0;
  while (q + 1 < jobs.n && (int)blockIdx.x >= jobs.j[q + 1].first) ++q;
  const TnSmallJob &a = jobs.j[q];
  const int tile = (int)blockIdx.x - a.first, m0 = tile / a.tiles_n * 16, n0 = tile % a.tiles_n * 16;
  const int m = min(m0 + (lane & 15), a.M - 1), n = min(n0 + (lane & 15), a.N - 1), g = lane >> 4;  // (lanes past the end are not stored)
  const float *const pa = a.A2 && m >= a.a_split ? a.A2 + (m - a.a_split) : a.A + m;
  const float *const pb = a.B + n;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = wid * 32; k0 < a.K; k0 += NW * 32) {
    f32x4 x[2], y[2];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = min(k0 + g * 8 + e, a.K - 1);
      x[e / 4][e % 4] = pa[(size_t)k * a.lda];
      y[e / 4][e % 4] = pb[(size_t)k * a.N];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool in = k0 + g * 8 + e < a.K;
      x[e / 4][e % 4] = in ? x[e / 4][e % 4] : 0.f;
      y[e / 4][e % 4] = in ? y[e / 4][e % 4] : 0.f;
    }
    const Frag3 fy = split8(y[0], y[1]);
    Frag3 fx[1];
    fx[0] = wid & 1 ? split8<true>(x[0], x[1]) : split8(x[0], x[1]);  // (odd sums run negated: mfma_split)
    f32x4 t[1];
    mfma_split<1>(t, fy, fx);
    acc += t[0];
  }
  *reinterpret_cast<f32x4 *>(&part[wid][lane * 4]) = wid & 1 ? -acc : acc;
  __syncthreads();
  const int e = threadIdx.x;
  if (e >= 256) return;
  float s = sum_in_pairs<NW>(part, e);
  // element e: lane e / 4, register e % 4, that is column (lane % 16) of A and 4 (lane / 16) + e % 4 of B
  const int cm = m0 + ((e >> 2) & 15), cn = n0 + (e >> 6) * 4 + (e & 3);
  if (cm >= a.M || cn >= a.N) return;
  if (!is_finite(s)) {
    const float *const px = a.A2 && cm >= a.a_split ? a.A2 + (cm - a.a_split) : a.A + cm;
    s = 0.f;
#pragma unroll 1
    for (int k = 0; k < a.K; ++k) s = fmaf(px[(size_t)k * a.lda], a.B[(size_t)k * a.N + cn], s);
  }
  const size_t at = (size_t)cm * a.N + cn;
  a.C[at] = s;
  if (a.W) a.W[at] -= jobs.lr * s;
}

namespace {

struct TnPlan { int mb, nb, tiles_m, tiles_n, splits; };

constexpr int kTnBlocks = 768;   // workgroups of a launch: three per compute unit, one resident round
constexpr int kTnMinRows = 64;   // per split
constexpr int kTnAlone = 512;    // rows per split from which a job is not batched

// Tile shape: the cheapest cover of the result.  A step of 32 depths costs a workgroup (in cycles, and what the
// matrix and vector pipes do hardly overlaps) 24 per 16 x 16 products, 2.75 per column that it splits, and a
// fixed part.  Where 128 x 128 tiles and depth chunks of 256 rows would leave most of the chip idle, tiles of at most
// 64 x 64: smaller chunks would store more in partial sums than they read.
void tn_tiles(int32_t M, int32_t N, int64_t K, TnPlan *b) {
  static const int mbs[2] = {128, 64}, nbs[4] = {128, 96, 64, 32};
  const bool shallow = (int64_t)((M + 127) / 128) * ((N + 127) / 128) * (K / 256) < kTnBlocks / 3;
  double best = 0.0;
  b->mb = 0;
  for (int mb : mbs)
    for (int nb : nbs) {
      if (shallow && (mb > 64 || nb > 64)) continue;
      const double cost = (double)((M + mb - 1) / mb) * ((N + nb - 1) / nb) * (24.0 * (mb / 16) * (nb / 16) + 2.75 * (mb + nb) + 200.0);
      if (b->mb == 0 || cost < best) {
        b->mb = mb;
        b->nb = nb;
        best = cost;
      }
    }
  b->tiles_m = (M + b->mb - 1) / b->mb;
  b->tiles_n = (N + b->nb - 1) / b->nb;
}

int tn_splits(int64_t K, int64_t chunk) { return (int)std::max<int64_t>(1, (K + chunk - 1) / chunk); }

// Product and sum in one launch?  It saves the launch of the sums, 3 to 4 us, and those of further tile shapes; a round of 512
// workgroups and 512 rows takes 1.7 to 2.3 us.  The line: three rounds, six where the products alone are two launches or more.
// Steps, general way / so, us: 64-16-8, 400 rows (one round) 29.5 / 24.9, 1000 (2) 32.0 / 29.2, 2000 (4) 36.0 / 35.9, 3000 (6) 43.8 / 47.3;
// 128-128-128-47, 400 rows 50.5 / 45.4, 1000 55.4 / 53.6, 2000 66.6 / 67.4; with several launches, mean aggregator 100-66-66-9, 400 rows 89.6 / 78.5,
// 2000 107 / 98, 3000 115 / 111, 5000 (10) 126 / 130, 300-512-512-100, 400 rows (4) 132 / 124, 1000 (8) 141 / 142.  Not where a
// gradient or the weights lie in the same memory as an operand: the other way has read all before it writes.
bool tn_small(const TnGemm *g, int32_t n, int launches, TnSmallJobs *out) {
  constexpr int kRound = 512;
  int64_t blocks = 0, rows = 0;
  for (int i = 0; i < n; ++i) {
    if (g[i].rows || g[i].k_dev || g[i].accumulate) return false;
    const int tiles_n = (g[i].N + 15) / 16;
    const int lda = g[i].A2 ? g[i].a_split : g[i].M;
    out->j[out->n++] = TnSmallJob{g[i].A, g[i].A2, g[i].B, g[i].C, g[i].lr > 0.f ? g[i].W : nullptr, g[i].M, g[i].N, g[i].K, g[i].a_split, lda, tiles_n,
                                  (int)blocks};
    if (g[i].lr > 0.f) out->lr = g[i].lr;
    blocks += (int64_t)((g[i].M + 15) / 16) * tiles_n;
    rows = std::max<int64_t>(rows, g[i].K);
  }
  out->blocks = (int)blocks;
  if (n == 0 || ((blocks + kRound - 1) / kRound) * ((rows + kRound - 1) / kRound) > (launches > 1 ? 6 : 3)) return false;
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < n; ++k) {
      const size_t result = (size_t)g[i].M * g[i].N, a = (size_t)g[k].K * out->j[k].lda;
      for (const float *w : {(const float *)g[i].C, (const float *)out->j[i].W})
        if (w && (overlap(w, result, g[k].A, a) || (g[k].A2 && overlap(w, result, g[k].A2, a)) || overlap(w, result, g[k].B, (size_t)g[k].K * g[k].N)))
          return false;
    }
  return true;
}

template <int MB, int NB>
void launch_tn(const TnJobs &jobs, unsigned blocks, hipStream_t s) {
  gemm_tn_kernel<MB, NB><<<blocks, 256, 0, s>>>(jobs);
}

}  // namespace

size_t gemm_tn_partials(int32_t M, int32_t N, int32_t K, int32_t K_other) {
  TnPlan b;
  tn_tiles(M, N, std::max(K, K_other), &b);
  const int64_t nt = (int64_t)b.tiles_m * b.tiles_n;
  const int64_t splits = std::min<int64_t>(std::max<int64_t>(1, kTnBlocks / nt), tn_splits(K, kTnMinRows));
  return (size_t)(splits * nt * b.mb * b.nb);
}

hipError_t gemm_tn(const TnGemm *g, int32_t n, const TnLoss &loss, hipStream_t s) {
  if (n > kMaxTnJobs) return hipErrorInvalidValue;
  TnPlan plan[kMaxTnJobs];
  int64_t depth[kMaxTnJobs];
  for (int i = 0; i < n; ++i) {
    if (g[i].accumulate) plan[i] = plan[i - 1];  // the two parts of one gradient have the same result tiles
    else tn_tiles(g[i].M, g[i].N, std::max<int64_t>(g[i].K, i + 1 < n && g[i + 1].accumulate ? g[i + 1].K : 0), &plan[i]);
    depth[i] = g[i].k_dev ? g[i].k_expected : g[i].K;
  }
  // A job that fills the chip with chunks of kTnAlone rows or more gets a launch of its own, its splits dealt
  // evenly over the XCDs.  The smaller jobs of one tile shape share a launch and the length of a chunk: the
  // smallest with which their workgroups are one resident round, so that all of them end together.
  bool alone[kMaxTnJobs];
  for (int i = 0; i < n; ++i) {
    const int64_t nt = (int64_t)plan[i].tiles_m * plan[i].tiles_n;
    int64_t splits = std::max<int64_t>(1, kTnBlocks / nt);
    if (splits >= 8) splits = splits / 8 * 8;
    alone[i] = depth[i] / splits >= kTnAlone;
    if (alone[i]) plan[i].splits = (int)splits;
  }
  auto same = [&](int i, int k) { return !alone[k] && !alone[i] && plan[k].mb == plan[i].mb && plan[k].nb == plan[i].nb; };
  {
    TnSmallJobs small{};
    int launches = 0;  // of the products, otherwise
    for (int i = 0; i < n; ++i) {
      bool first = true;
      for (int k = 0; k < i; ++k) first &= !same(k, i);
      launches += first;
    }
    if (tn_small(g, n, launches, &small)) {
      small.loss = loss;
      gemm_tn_small_kernel<<<(unsigned)(small.blocks + (loss.out ? 1 : 0)), kTnSmallWaves * kWave, 0, s>>>(small);
      return hipGetLastError();
    }
  }
  for (int i = 0; i < n; ++i) {
    if (alone[i]) continue;
    auto blocks = [&](int64_t chunk) {
      int64_t b = 0;
      for (int k = 0; k < n; ++k)
        if (same(i, k)) b += (int64_t)plan[k].tiles_m * plan[k].tiles_n * tn_splits(depth[k], chunk);
      return b;
    };
    int64_t lo = kTnMinRows, hi = (int64_t)1 << 31;  // blocks(hi): one split each
    while (lo < hi) {
      const int64_t mid = (lo + hi) / 2;
      if (blocks(mid) <= kTnBlocks) hi = mid; else lo = mid + 1;
    }
    plan[i].splits = tn_splits(depth[i], lo);
  }
  TnSums sums{};
  for (int i = 0; i < n; ++i) {
    const int nt = plan[i].tiles_m * plan[i].tiles_n;
    if (g[i].accumulate) {
      TnSum &t = sums.j[sums.n - 1];
      t.partials2 = g[i].partials;
      t.splits2 = plan[i].splits;
      continue;
    }
    TnSum &t = sums.j[sums.n++];
    t = TnSum{g[i].partials, nullptr, g[i].C, g[i].lr > 0.f ? g[i].W : nullptr, g[i].M, g[i].N, plan[i].mb / 32, plan[i].nb / 32,
              plan[i].tiles_n, nt, plan[i].splits, 0, sums.blocks};
    if (g[i].lr > 0.f) sums.lr = g[i].lr;
    sums.blocks += nt * (plan[i].mb * plan[i].nb / 256);
  }
  bool done[kMaxTnJobs] = {};
  for (int i = 0; i < n; ++i) {
    if (done[i]) continue;
    TnJobs jobs{};
    int blocks = 0;
    for (int k = i; k < n; ++k) {
      if (k != i && (done[k] || !same(i, k))) continue;
      done[k] = true;
      const int nt = plan[k].tiles_m * plan[k].tiles_n;
      jobs.j[jobs.n++] = TnJob{g[k].A, g[k].A2, g[k].B, g[k].rows, g[k].k_dev, g[k].partials, g[k].M, g[k].N, g[k].K, g[k].a_split,
                               g[k].A2 ? g[k].a_split : g[k].M, plan[k].tiles_n, nt, plan[k].splits, blocks};
      blocks += nt * ((plan[k].splits + 7) / 8 * 8);  // every job starts on XCD 0
    }
#define BNS_TN(MB_, NB_) if (plan[i].mb == MB_ && plan[i].nb == NB_) launch_tn<MB_, NB_>(jobs, (unsigned)blocks, s)
    BNS_TN(128, 128); BNS_TN(128, 96); BNS_TN(128, 64); BNS_TN(128, 32);
    BNS_TN(64, 128); BNS_TN(64, 96); BNS_TN(64, 64); BNS_TN(64, 32);
#undef BNS_TN
  }
  bool many = false;
  for (int i = 0; i < sums.n; ++i) many |= std::max(sums.j[i].splits, sums.j[i].splits2) > 32;
  sums.loss = loss;
  const unsigned blocks = (unsigned)(sums.blocks + (loss.out ? 1 : 0));
  if (blocks == 0) return hipSuccess;
  if (many) gemm_tn_reduce_kernel<16><<<blocks, 1024, 0, s>>>(sums);
  else gemm_tn_reduce_kernel<4><<<blocks, 256, 0, s>>>(sums);
  return hipGetLastError();
}

}  // namespace bns
