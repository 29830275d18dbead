// The forward product H = [A | A2] W (Eq. 2) on the fp32 matrix instruction, v_mfma_f32_32x32x2_f32.
//
// The forward chain decides which hidden units a ReLU switches on, and a unit within rounding of
// zero is switched by another order of summation.  So every forward product of a hidden layer, whatever its kernel, adds
// the same terms in the same order: a chain over depth pairs (0,1), (2,3), ... from zero.  The last layer's and the backward
// products have no such decision behind them and run faster on split bf16 operands (gemm.hip).
//
// A workgroup of 4 wavefronts walks row tiles of 128; a wavefront owns 32 rows and NC column tiles of
// 32.  Its rows come straight from global memory: a lane reads four consecutive depths of its row, and
// a swap of wavefront halves per pair of registers turns the eight depths of the two halves into the
// operands of four instructions in depth order.  The weights, packed once per step as operand fragments,
// are copied from L2 into a double-buffered LDS tile, one 32-deep step ahead, across row tiles as well (those of a
// product of a single step once, to stay): one 16-byte LDS read feeds four instructions, and the matrix pipe is what is left
// to wait for.  The weights are the second operand of the instruction: a lane ends up with a column, and a wavefront stores
// 128 consecutive bytes of a row (with four columns per lane, 32-byte pieces of 32 rows: 32 -> 128 on 578125 rows 94 us, 79).
// What bounds it: the matrix pipe where the depth is large, the stores where it is a step or two.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"
#include "split_bf16.hpp"

namespace bns {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int kF32Step = 4096;  // bytes of the packed weights of one 32-deep step and one column tile of 32

struct F32Args {
  RowsF32 g;
  int T, S, nblk;  // column tiles of 32, depth steps of 32, column blocks
};

// REC: the rows of A are followed by the ones that g.rec names (a second result, row tiles of its own).
template <int NC, bool ACC, bool REC>
__global__ void __launch_bounds__(256, NC > 2 ? 3 : 4) gemm_rows_f32_kernel(const F32Args a) {
  constexpr int kRows = 128;
  __shared__ __attribute__((aligned(16))) char Bs[2][NC * kF32Step];
  const RowsF32 &p = a.g;
  const int M = p.M, M2 = REC ? min(p.M2, *p.m2_dev) : 0;
  // workgroup b runs on XCD b % 8: the column blocks of one row tile follow each other on one XCD
  const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
  const int nb = q % a.nblk, stride = (gridDim.x / (8 * a.nblk)) * 8;
  const int t0 = nb * NC;
  int tile = (q / a.nblk) * 8 + x;
  const int n_first = (M + kRows - 1) / kRows;  // row tiles of the first result
  const int n_tiles = n_first + (M2 + kRows - 1) / kRows;
  if (tile >= n_tiles) return;

  const int lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int S = a.S;
  const bool two = p.A2 != nullptr;  // then a_split % 16 == 0

  f32x4 ar[4];
  const float *row_a, *row_a2;
  float row_scale = 1.f;  // REC: of the row whose values ar holds
  auto set_rows = [&](int tl) {
    int row = min(M - 1, tl * kRows + wid * 32 + l32);  // rows past the end are not stored
    const float *A = p.A;
    if constexpr (REC) {
      row_scale = 1.f;
      if (tl >= n_first) {
        const int2 r = p.rec[min(M2 - 1, (tl - n_first) * kRows + wid * 32 + l32)];
        row = r.x;
        row_scale = __int_as_float(r.y);
        A = p.A_rec;
      }
    }
    row_a = A + (size_t)row * p.lda;
    row_a2 = two ? p.A2 + (size_t)row * p.lda - p.a_split : nullptr;
  };
  auto load_a = [&](int s) {
    const float *src[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = s * 32 + j * 8 + hi * 4;
      src[j] = (two && k >= p.a_split ? row_a2 : row_a) + k;
    }
    if ((s + 1) * 32 <= p.K) {
#pragma unroll
      for (int j = 0; j < 4; ++j) ar[j] = *reinterpret_cast<const f32x4u *>(src[j]);
    } else if ((p.K & 3) == 0) {  // pieces in or out as a whole
#pragma unroll
      for (int j = 0; j < 4; ++j)
        ar[j] = s * 32 + j * 8 + hi * 4 < p.K ? *reinterpret_cast<const f32x4u *>(src[j]) : f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = s * 32 + j * 8 + hi * 4;
        if (k + 4 <= p.K) ar[j] = *reinterpret_cast<const f32x4u *>(src[j]);
        else
#pragma unroll
          for (int e = 0; e < 4; ++e) ar[j][e] = k + e < p.K ? src[j][e] : 0.f;
      }
    }
  };
  const unsigned lds0 = lds_offset_of(&Bs[0][0]);
  const int nt = min(NC, a.T - t0);
  auto load_b = [&](int s, int buf) {  // pieces of 1 KB, dealt to the four wavefronts
    const char *src = static_cast<const char *>(p.Bp) + (size_t)(s * a.T + t0) * kF32Step + lane * 16;
    for (int c = wid; c < nt * 4; c += 4) lds_dma16(src + c * 1024, lds0 + buf * (NC * kF32Step) + c * 1024);
  };

  f32x16 acc[NC];
  auto clear = [&]() {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[c][i] = 0.f;
  };
  const bool stay = S == 1;  // the weights of a single step stay in LDS for all tiles
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
    if (!stay) {
      lds_dma_wait();
      __syncthreads();  // this step's weights are in LDS, and everybody is done with the other buffer
    }
    if constexpr (REC) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) ar[j][e] *= row_scale;
    }
    // depths 8 j + 4 hi + 0..3 -> pairs (8 j + 2 i, 8 j + 2 i + 1) in the two halves
    float op[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const u32x2 w = __builtin_amdgcn_permlane32_swap(__float_as_uint(ar[j][2 * h]), __float_as_uint(ar[j][2 * h + 1]),
                                                         false, false);
        op[j][h] = __uint_as_float(w[0]);
        op[j][2 + h] = __uint_as_float(w[1]);
      }
    const bool last = s + 1 == S;
    const int ntile = last ? tile + stride : tile, ns = last ? 0 : s + 1;
    if (ntile < n_tiles) {
      if (last) set_rows(ntile);
      if (!stay) load_b(ns, buf ^ 1);
      load_a(ns);
    }
    const char *bs = &Bs[buf][0] + lane * 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x4 b[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) b[c] = *reinterpret_cast<const f32x4 *>(bs + c * kF32Step + j * 1024);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(op[j][i], b[c][i], acc[c], 0, 0, 0);
    }
    buf = stay ? ns : buf ^ 1;
    if (last) {
      // lane: column 32 c + l32; register 4 q + e of tile c: row 8 q + 4 hi + e of the wavefront's 32
      const bool second = REC && tile >= n_first;
      const int row0 = (second ? tile - n_first : tile) * kRows + wid * 32, rows = (second ? M2 : M) - row0;
      const int n_end = p.pad ? p.ldc : p.N;  // pad: the packed weights are zero there
      float *const dst = (second ? p.C_rec : p.C) + (size_t)row0 * p.ldc;
      auto store = [&](auto full) {  // full: all 32 rows are there
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int col = (t0 + c) * 32 + l32;
          if (NC > 1 && col >= n_end) continue;
          const bool in = NC > 1 || col < n_end;
          const unsigned at = (unsigned)(hi * 4 * p.ldc + col) * 4u;  // bytes
          auto each = [&](int q, f32x4 &v, auto f) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (in && (decltype(full)::value || q * 8 + hi * 4 + e < rows)) v[e] = f(reinterpret_cast<float *>(reinterpret_cast<char *>(dst + (size_t)(q * 8 + e) * p.ldc) + at), v[e]);
          };
          // Where the tiles are few and small, latency counts: all lanes draw for the dropout, those past the last column too (a
          // wavefront with two of its columns active took three times as long over it: 512 rows, 64 -> 66 15.2 us, 10.0), and what
          // is added to is read before the first store, which a later load would wait for (1211 rows, 300 -> 300 29.6 us, 27.4).
          // With more tiles per wavefront neither pays (60000 rows, 130 -> 130 95 us, 104).
          constexpr bool kOldFirst = ACC && NC == 1;
          f32x4 old[4];
          if constexpr (kOldFirst)
#pragma unroll
            for (int q = 0; q < 4; ++q) each(q, old[q], [](const float *d, float) { return *d; });
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f32x4 v = {acc[c][4 * q], acc[c][4 * q + 1], acc[c][4 * q + 2], acc[c][4 * q + 3]};
            if constexpr (kOldFirst) v += old[q];
            else if constexpr (ACC) each(q, v, [](const float *d, float x) { return x + *d; });
            if (p.relu) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
              if (p.drop.scale != 0.f) {
#pragma unroll 1
                for (int e = 0; e < 4; ++e) {
                  const float y = dropout_keeps(p.drop, row0 + q * 8 + hi * 4 + e, col) ? v[0] * p.drop.scale : 0.f;
                  v = f32x4{v[1], v[2], v[3], y};
                }
              }
            }
            each(q, v, [](float *d, float x) { return *d = x; });
          }
        }
      };
      if (rows >= 32) store(std::true_type{});
      else store(std::false_type{});
      if (ntile >= n_tiles) break;
      clear();
      tile = ntile;
    }
    s = ns;
  }
}

hipError_t gemm_rows_f32(const RowsF32 &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.ldc < g.N || (g.pad && (g.ldc > (g.N + 3) / 4 * 4 || g.relu || g.accumulate)) || (g.A2 && g.a_split % 16 != 0) ||
      (g.rec && (g.A2 || g.accumulate || g.relu || !g.m2_dev)))
    return hipErrorInvalidValue;
  F32Args a;
  a.g = g;
  a.T = (g.N + 31) / 32;
  a.S = (g.K + 31) / 32;
  // Up to 4 column tiles per wavefront, evenly dealt; fewer where that leaves the chip short of workgroups.  Three or four are held to three
  // workgroups per compute unit, which spills nothing (four: 26 registers of the four-tile kernel, 423 us instead of 369 for
  // 89625 x 512 x 512).  A product of a single step is bound by its stores: two tiles and a workgroup per row tile
  // (578125 rows, 16 -> 172: 126 us walked with four tiles, 103; 32 -> 128: 82, 73).
  const int64_t row_tiles = (g.M + 127) / 128 + (g.rec ? (g.m2_expected + 127) / 128 : 0);
  a.nblk = a.S == 1 ? (a.T + 1) / 2 : (a.T + 3) / 4;
  while (row_tiles * a.nblk < 512 && a.nblk < a.T) a.nblk = std::min(a.nblk * 2, a.T);
  int nc = (a.T + a.nblk - 1) / a.nblk;
  a.nblk = (a.T + nc - 1) / nc;
  // Or fewer yet, where all workgroups are still resident and the compute unit with the most tiles has a tenth less of them (us, by the rules
  // above / so: 10000 rows and 7500 by record, 602 -> 130, 411 workgroups of two tiles 52.0 / 685 of one 45.7; 15000 and 2000, 300 -> 130, 402 of two
  // 30.0 / 670 of one 25.9; 40000, 130 -> 130, 626 of three 34.2 / 939 of two 31.7).  With as many on the fullest unit the wider ones
  // read their rows less often: 20011, 602 -> 130, 471 of two 50.4 / 785 of one 55.1; 29125 and 19800, 602 -> 256, 766 of four 131 / 1532 of two 141.
  auto most = [&](int nblk) { return (row_tiles * nblk + 255) / 256 * ((a.T + nblk - 1) / nblk); };  // on one of 256 units
  if (a.S > 1)
    for (int n = a.nblk + 1; n <= a.T; ++n)
      if (row_tiles * n <= ((a.T + n - 1) / n > 2 ? 768 : 1024) && 10 * most(n) <= 9 * most(a.nblk)) a.nblk = n;
  nc = (a.T + a.nblk - 1) / a.nblk;
  a.nblk = (a.T + nc - 1) / nc;
  int64_t octets = (row_tiles + 7) / 8;
  if (a.S > 1) octets = std::min<int64_t>(octets, std::max<int64_t>(1, (nc > 2 ? 768 : 1024) / (8 * a.nblk)));
  const unsigned grid = (unsigned)(octets * 8 * a.nblk);
#define BNS_ROWS_F32(NC)                                                          \
  do {                                                                          \
    if (g.accumulate) gemm_rows_f32_kernel<NC, true, false><<<grid, 256, 0, s>>>(a); \
    else if (g.rec) gemm_rows_f32_kernel<NC, false, true><<<grid, 256, 0, s>>>(a);   \
    else gemm_rows_f32_kernel<NC, false, false><<<grid, 256, 0, s>>>(a);             \
  } while (0)
  switch (nc) {
    case 1: BNS_ROWS_F32(1); break;
    case 2: BNS_ROWS_F32(2); break;
    case 3: BNS_ROWS_F32(3); break;
    default: BNS_ROWS_F32(4); break;
  }
#undef BNS_ROWS_F32
  return hipGetLastError();
}

}  // namespace bns
