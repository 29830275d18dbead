// The backward products of the update (Eq. 2) on the matrix cores: fp32 operands and results, products by
// three-way bf16 splitting (split_bf16.hpp).
//
//   gemm_rows   C = A B   dA = dZ W^T: a tall A [M, K] times a weight matrix, which pack_weights has
//               split and laid out as operand fragments
//   gemm_tn     C = [A | A2]^T B  weight gradient dW = A^T dZ, the depth (rows) split over the chip
//
// gemm_rows: a workgroup of 4 wavefronts walks row tiles; a wavefront owns 16 R rows and NC column
// tiles of 16.  Its rows come straight from global memory into the operand layout (a lane reads two
// 16-byte pieces of its row per 32-deep step, four lanes of a row 64 contiguous bytes) and are split in
// registers, each element once.  The packed weights of a step go from L2 straight into a
// double-buffered LDS tile shared by the four wavefronts, one step ahead, across row tiles as well.
// The weight fragment is the first operand of the instruction, so a lane ends up with four
// consecutive columns of one row and stores 16 bytes.
//
// gemm_tn: a thread reads 16-byte pieces of eight consecutive-depth rows of one operand, which makes
// it hold eight depths of four columns: after the split each column's eight values are one 16-byte
// fragment entry in LDS.  The partial tiles are stored as the accumulators lie in the registers;
// one kernel adds them in a fixed order and puts the elements where they belong.
//
// What bounds them: the 128-wide products move 1 KB per row for 32 k flops and are bound by memory,
// the 512-wide ones by the matrix cores (6 of 16 instruction slots per fp32 product).
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"
#include "split_bf16.hpp"

namespace bns {

// ---- packed weights -----------------------------------------------------------------------------
// Operand fragments, 1 KB each (64 lanes x 16 bytes), zero outside the matrix.
//   split: of W [N, K] transposed, for gemm_rows.  For depth step s of 32 and column tile t of 16, at
//     ((s * tiles + t) * 3 + piece) KB, lane l's 8 values are column 16 t + l % 16 at the depths
//     32 s + 16 (e / 4) + 4 (l / 16) + e % 4, e = 0..7, negated in even steps (mfma_split)
//   fp32: of W [K, N], for gemm_rows_f32.  For depth step s of 32, column tile t of 32 and depth group j of 8, at
//     ((s * tiles + t) * 4 + j) KB, lane l's 4 values are column 32 t + l % 32 at the depths
//     32 s + 8 j + 2 i + l / 32, i = 0..3
__host__ __device__ static inline int k_steps(int K) { return (K + 31) / 32; }
__host__ __device__ static inline int col_tiles(int N) { return (N + 15) / 16; }
__host__ __device__ static inline int pack_units(const PackJob &j) {  // a wavefront's work: one fragment set
  return k_steps(j.K) * (j.split ? col_tiles(j.N) : (j.N + 31) / 32);
}

size_t packed_bytes(int32_t K, int32_t N) { return (size_t)k_steps(K) * col_tiles(N) * kFragSet; }
size_t packed_bytes_f32(int32_t K, int32_t N) { return (size_t)k_steps(K) * ((N + 31) / 32) * 4096; }

struct PackJobs {
  PackJob j[kMaxPackJobs];
  int n;
};

__global__ void __launch_bounds__(256) pack_weights_kernel(const PackJobs jobs) {
  int u = blockIdx.x * 4 + (threadIdx.x >> 6);
  int q = 0;
  for (; q < jobs.n; ++q) {
    const int units = pack_units(jobs.j[q]);
    if (u < units) break;
    u -= units;
  }
  if (q == jobs.n) return;
  const PackJob &job = jobs.j[q];
  const int lane = lane_id();
  if (job.split) {
    const int T = col_tiles(job.N), s = u / T, t = u % T;
    const int n = t * 16 + (lane & 15), g = lane >> 4;
    f32x4 v[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = s * 32 + j * 16 + g * 4 + e;
        v[j][e] = k < job.K && n < job.N ? job.W[(size_t)n * job.K + k] : 0.f;
      }
    const Frag3 f = s % 2 == 0 ? split8<true>(v[0], v[1]) : split8(v[0], v[1]);
    char *out = static_cast<char *>(job.out) + (size_t)u * kFragSet + lane * 16;
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<bf16x8 *>(out + p * kFragBytes) = f.p[p];
  } else {
    const int T = (job.N + 31) / 32, s = u / T, t = u % T;
    const int n = t * 32 + (lane & 31);
    char *out = static_cast<char *>(job.out) + (size_t)u * 4096 + lane * 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = s * 32 + j * 8 + i * 2 + (lane >> 5);
        v[i] = k < job.K && n < job.N ? job.W[(size_t)k * job.N + n] : 0.f;
      }
      *reinterpret_cast<f32x4 *>(out + j * 1024) = v;
    }
  }
}

hipError_t pack_weights(const PackJob *jobs, int32_t n, hipStream_t s) {
  for (int32_t i0 = 0; i0 < n; i0 += kMaxPackJobs) {
    PackJobs pj;
    pj.n = std::min<int32_t>(kMaxPackJobs, n - i0);
    int64_t units = 0;
    for (int i = 0; i < pj.n; ++i) {
      pj.j[i] = jobs[i0 + i];
      units += pack_units(pj.j[i]);
    }
    if (units) pack_weights_kernel<<<(unsigned)((units + 3) / 4), 256, 0, s>>>(pj);
  }
  return hipGetLastError();
}

// ---- rows x packed weights ------------------------------------------------------------------------
struct RowsArgs {
  RowsGemm g;
  int T, S, nblk;  // column tiles, depth steps, column blocks
};

enum RowsEpilogue { kPlain = 0, kMask = 1, kPair = 2 };

template <int R, int NC, int EPI>
__global__ void __launch_bounds__(256, R * NC > 8 ? 3 : 4) gemm_rows_kernel(const RowsArgs a) {
  constexpr int kRows = 64 * R;  // rows of a workgroup's tile
  __shared__ __attribute__((aligned(16))) char Bs[2][NC * kFragSet];
  const RowsGemm &p = a.g;
  const int M = p.m_dev ? min(p.M, *p.m_dev) : p.M;
  // workgroup b runs on XCD b % 8: the column blocks of one row tile follow each other on one XCD, so
  // that they find its rows in that XCD's L2
  const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
  const int nb = q % a.nblk, stride = (gridDim.x / (8 * a.nblk)) * 8;
  const int t0 = nb * NC;
  int tile = (q / a.nblk) * 8 + x;
  const int n_tiles = (M + kRows - 1) / kRows;
  if (tile >= n_tiles) return;

  const int lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int S = a.S;

  f32x4 ar[R][2];
  const float *row_a[R];
  auto set_rows = [&](int tl) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = min(M - 1, tl * kRows + wid * 16 * R + r * 16 + l16);  // rows past the end are not stored
      row_a[r] = p.A + (size_t)row * p.K;
    }
  };
  auto load_a = [&](int s) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int k = s * 32 + j * 16 + g * 4;
      if ((s + 1) * 32 <= p.K) {
#pragma unroll
        for (int r = 0; r < R; ++r) ar[r][j] = *reinterpret_cast<const f32x4u *>(row_a[r] + k);
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int e = 0; e < 4; ++e) ar[r][j][e] = k + e < p.K ? row_a[r][k + e] : 0.f;
      }
    }
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
  set_rows(tile);
  load_b(0, 0);
  load_a(0);
  clear();
  int buf = 0;
  for (int s = 0;;) {
    Frag3 fa[R];
    lds_dma_wait();
    __syncthreads();  // this step's weights are in LDS, and everybody is done with the other buffer
#pragma unroll
    for (int r = 0; r < R; ++r) fa[r] = split8(ar[r][0], ar[r][1]);
    const bool last = s + 1 == S;
    const int ntile = last ? tile + stride : tile, ns = last ? 0 : s + 1;
    if (ntile < n_tiles) {
      if (last) set_rows(ntile);
      load_b(ns, buf ^ 1);
      load_a(ns);
    }
    const char *bs = &Bs[buf][0] + lane * 16;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Frag3 fb;
#pragma unroll
      for (int i = 0; i < 3; ++i) fb.p[i] = *reinterpret_cast<const bf16x8 *>(bs + c * kFragSet + i * kFragBytes);
      mfma_split<R>(acc[c], fb, fa, s & 1 ? 1.f : -1.f);
    }
    buf ^= 1;
    if (last) {
      // lane: row l16 of the row tile, columns 16 c + 4 g .. + 3
      const int n_end = p.N, col0 = t0 * 16 + g * 4;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int row = tile * kRows + wid * 16 * R + r * 16 + l16;
        if (row >= M) continue;
        const size_t at = (size_t)row * p.ldc + col0;
        float *const dst = p.C + at;
        float *const dst2 = EPI == kPair ? p.C2 + at - p.c_split : nullptr;  // c_split % 4 == 0
        const float *const ms = EPI == kMask ? p.mask + at : nullptr;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int left = n_end - (col0 + c * 16);  // columns from this lane's first one to the end
          f32x4 v = acc[c][r];
          if constexpr (EPI == kMask) {
            f32x4 m = {0.f, 0.f, 0.f, 0.f};
            if (left >= 4) m = *reinterpret_cast<const f32x4u *>(ms + c * 16);
            else
#pragma unroll
              for (int e = 0; e < 3; ++e)
                if (e < left) m[e] = ms[c * 16 + e];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = m[e] > 0.f ? v[e] * p.alpha : 0.f;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= p.alpha;
          }
          float *const d = (EPI == kPair && col0 + c * 16 >= p.c_split ? dst2 : dst) + c * 16;
          if (left >= 4) *reinterpret_cast<f32x4u *>(d) = v;
          else
#pragma unroll
            for (int e = 0; e < 3; ++e)
              if (e < left) d[e] = v[e];
        }
      }
      if (ntile >= n_tiles) break;
      clear();
      tile = ntile;
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
  if (a.g.C2) launch_rows<R, kPair>(a, nc, grid, s);
  else if (a.g.mask) launch_rows<R, kMask>(a, nc, grid, s);
  else launch_rows<R, kPlain>(a, nc, grid, s);
}

hipError_t gemm_rows(const RowsGemm &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.C2 ? g.c_split % 4 != 0 || g.ldc < g.c_split || g.N > 2 * g.c_split : g.ldc < g.N) return hipErrorInvalidValue;
  if (g.C2 && g.mask) return hipErrorInvalidValue;
  RowsArgs a;
  a.g = g;
  a.T = col_tiles(g.N);
  a.S = k_steps(g.K);
  // Up to 8 column tiles per wavefront, evenly dealt.  Where that leaves the chip short of workgroups
  // (three fit a compute unit), smaller tiles: first half the rows, then half the columns.
  constexpr int kWanted = 512;
  a.nblk = (a.T + 7) / 8;
  int R = 2;
  auto groups = [&]() { return (int64_t)((g.M + 64 * R - 1) / (64 * R)) * a.nblk; };
  if (groups() < kWanted) R = 1;
  while (groups() < kWanted && a.nblk * 2 <= a.T) a.nblk *= 2;
  int nc = (a.T + a.nblk - 1) / a.nblk;
  a.nblk = (a.T + nc - 1) / nc;
  const int64_t row_tiles = (g.M + 64 * R - 1) / (64 * R);
  // a grid of whole octets of row tiles, every column block of each; the tiles past one resident round are walked
  int64_t octets = std::min<int64_t>((row_tiles + 7) / 8, std::max<int64_t>(1, 768 / (8 * a.nblk)));
  const unsigned grid = (unsigned)(octets * 8 * a.nblk);
  if (R == 2) launch_rows<2>(a, nc, grid, s);
  else launch_rows<1>(a, nc, grid, s);
  return hipGetLastError();
}

// ---- transposed product, depth split over the chip -----------------------------------------------
struct TnArgs {
  const float *A, *A2, *B;
  int M, N, K, a_split, lda;
  const int *k_dev;
  float *partials;
  int tiles_m, tiles_n, splits;
};

// Bytes between the fragment sets of neighbouring 16-column tiles in LDS: 64 more than a set, so
// that the eight lanes that store together (four columns of two tiles) hit different banks.
constexpr int kTnTile = kFragSet + 64;

template <int MB, int NB>
__global__ void __launch_bounds__(256, 3) gemm_tn_kernel(const TnArgs a) {
  constexpr int KS = MB + NB > 128 ? 32 : 64;          // depth of a step: keeps all 256 threads loading
  constexpr int TM = MB / 16, TN = NB / 16, TILES = TM + TN;
  constexpr int GA = MB / 4, GB = NB / 4;              // 4-column groups of the two operands
  constexpr int KG = KS / 8;                           // groups of eight depths
  constexpr int MT = TM / 2, NT = TN / 2;              // 16 x 16 tiles of a wavefront (2 x 2 wavefronts)
  static_assert((GA + GB) * KG <= 256, "one load unit per thread");
  __shared__ __attribute__((aligned(16))) char lds[(KS / 32) * TILES * kTnTile];

  const int nt = a.tiles_m * a.tiles_n;
  int tile, split;
  if (a.splits % 8 == 0) {  // the tiles of one depth chunk follow each other on one XCD
    const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
    tile = q % nt;
    split = (q / nt) * 8 + x;
  } else {
    tile = blockIdx.x % nt;
    split = blockIdx.x / nt;
  }
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
  int ld, cols;  // columns in range at src (0..4)
  if (is_b) {
    src = a.B + n0 + c4 * 4;
    ld = a.N;
    cols = a.N - (n0 + c4 * 4);
  } else {
    int c = m0 + c4 * 4;
    src = a.A + c;
    ld = a.lda;
    cols = (a.A2 ? a.a_split : a.M) - c;
    if (a.A2 && cols <= 0) {
      src = a.A2 + c - a.a_split;
      cols = a.M - c;
    }
  }
  const bool straddle = !is_b && a.A2 && cols > 0 && cols < 4;  // a_split % 4 != 0: one group takes from both
  const int row_of_a2 = straddle ? m0 + c4 * 4 - a.a_split : 0;
  cols = straddle ? min(4, a.M - (m0 + c4 * 4)) : max(0, min(4, cols));
  f32x4 v[8];
  auto load = [&](int k0) {
    const int k = k0 + kg * 8;
    if (!active) return;
    if (cols == 4 && !straddle && k + 8 <= k_end) {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const f32x4u *>(src + (size_t)(k + j) * ld);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float xv = 0.f;
          if (e < cols && k + j < k_end)
            xv = straddle && row_of_a2 + e >= 0 ? a.A2[(size_t)(k + j) * ld + row_of_a2 + e] : src[(size_t)(k + j) * ld + e];
          v[j][e] = xv;
        }
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
  if (k_begin < k_end) load(k_begin);
  for (int k0 = k_begin; k0 < k_end; k0 += KS) {
    __syncthreads();  // the previous step's fragments have been read
    if (active) {
      if (neg) stage(std::true_type{});
      else stage(std::false_type{});
    }
    __syncthreads();
    if (k0 + KS < k_end) load(k0 + KS);
#pragma unroll
    for (int ks = 0; ks < KS / 32; ++ks) {
      const char *base = lds + (size_t)ks * TILES * kTnTile + lane * 16;
      Frag3 fm[MT];
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          fm[i].p[p] = *reinterpret_cast<const bf16x8 *>(base + (wm * MT + i) * kTnTile + p * kFragBytes);
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        Frag3 fn;
#pragma unroll
        for (int p = 0; p < 3; ++p)
          fn.p[p] = *reinterpret_cast<const bf16x8 *>(base + (TM + wn * NT + j) * kTnTile + p * kFragBytes);
        mfma_split<MT>(acc[j], fn, fm);
      }
    }
  }
  float *out = a.partials + (size_t)(split * nt + tile) * (MB * NB) + (size_t)wid * (MT * NT * 256) + lane * 4;
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) *reinterpret_cast<f32x4 *>(out + (j * MT + i) * 256) = split & 1 ? -acc[j][i] : acc[j][i];
}

// C = (C +) sum over the splits, in a fixed order; optionally W -= lr * C (the update step of
// Algorithm 1 takes its gradient from the registers).  A workgroup owns one 16 x 16 accumulator
// tile: NW wavefronts add every NW-th partial of it, then their sums are added in ascending order.
struct TnReduce {
  const float *partials;
  float *C, *W;
  float lr;
  int M, N, tiles_n, nt, splits;
  bool accumulate;
};

template <int MB, int NB, int NW>
__global__ void __launch_bounds__(NW * 64) gemm_tn_reduce_kernel(const TnReduce a) {
  constexpr int MT = MB / 32, NT = NB / 32, F = MB * NB / 256;
  __shared__ float part[NW][256];
  const int lane = lane_id(), wid = threadIdx.x >> 6;
  const int tile = blockIdx.x / F, f = blockIdx.x % F;
  const size_t stride = (size_t)a.nt * (MB * NB);
  const float *in = a.partials + (size_t)tile * (MB * NB) + f * 256 + lane * 4;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 4;
  for (int z0 = wid; z0 < a.splits; z0 += U * NW) {
    f32x4 x[U];
#pragma unroll
    for (int i = 0; i < U; ++i)
      x[i] = z0 + i * NW < a.splits ? *reinterpret_cast<const f32x4 *>(in + (size_t)(z0 + i * NW) * stride) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < U; ++i) sum += x[i];
  }
  *reinterpret_cast<f32x4 *>(&part[wid][lane * 4]) = sum;
  __syncthreads();
  const int e = threadIdx.x;
  if (e >= 256) return;
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) s += part[w][e];
  // element e: lane e / 4, register e % 4; its slots in the two 16-column tiles are 4 (lane / 16) + e % 4
  // (columns of B) and lane % 16 (columns of A), slot q standing for column 4 (q % 4) + q / 4
  const int l = e >> 2, w4 = f / (MT * NT), ji = f % (MT * NT);
  const int j = ji / MT, i = ji % MT, sa = l & 15;
  const int m = (tile / a.tiles_n) * MB + ((w4 >> 1) * MT + i) * 16 + 4 * (sa & 3) + (sa >> 2);
  const int n = (tile % a.tiles_n) * NB + ((w4 & 1) * NT + j) * 16 + 4 * (e & 3) + (l >> 4);
  if (m >= a.M || n >= a.N) return;
  const size_t at = (size_t)m * a.N + n;
  if (a.accumulate) s += a.C[at];
  a.C[at] = s;
  if (a.W) a.W[at] -= a.lr * s;
}

namespace {

struct TnPlan { int mb, nb, tiles_m, tiles_n, splits; };

// Tile shape: the one that pads the result least; among equals the larger one (an operand is read
// once per tile of the other).  Splits: three workgroups per compute unit, at least 64 rows each.
TnPlan tn_plan(int32_t M, int32_t N, int32_t K) {
  static const int mbs[2] = {128, 64}, nbs[4] = {128, 96, 64, 32};
  TnPlan b{};
  int64_t best = 0;
  for (int mb : mbs)
    for (int nb : nbs) {
      const int64_t area = (int64_t)((M + mb - 1) / mb * mb) * ((N + nb - 1) / nb * nb);
      if (b.mb == 0 || area * 10 < best * 9) {
        b.mb = mb;
        b.nb = nb;
        best = area;
      }
    }
  b.tiles_m = (M + b.mb - 1) / b.mb;
  b.tiles_n = (N + b.nb - 1) / b.nb;
  const int nt = b.tiles_m * b.tiles_n;
  int64_t splits = std::max(1, 768 / nt);
  splits = std::max<int64_t>(1, std::min<int64_t>(splits, (K + 63) / 64));
  if (splits >= 8) splits = splits / 8 * 8;
  b.splits = (int)splits;  // trailing splits may be empty: they store zeros
  return b;
}

template <int MB, int NB>
void launch_tn(const TnArgs &a, const TnReduce &r, hipStream_t s) {
  gemm_tn_kernel<MB, NB><<<(unsigned)(r.nt * a.splits), 256, 0, s>>>(a);
  const unsigned blocks = (unsigned)(r.nt * (MB * NB / 256));
  if (a.splits > 32) gemm_tn_reduce_kernel<MB, NB, 16><<<blocks, 1024, 0, s>>>(r);
  else gemm_tn_reduce_kernel<MB, NB, 4><<<blocks, 256, 0, s>>>(r);
}

}  // namespace

size_t gemm_tn_partials(int32_t M, int32_t N, int32_t K) {
  const TnPlan b = tn_plan(M, N, K);
  return (size_t)b.splits * b.tiles_m * b.tiles_n * b.mb * b.nb;
}

hipError_t gemm_tn(const TnGemm &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  const TnPlan b = tn_plan(g.M, g.N, g.K);
  TnArgs a{g.A, g.A2, g.B, g.M, g.N, g.K, g.a_split, g.A2 ? g.a_split : g.M, g.k_dev, g.partials, b.tiles_m, b.tiles_n, b.splits};
  TnReduce r{g.partials, g.C, g.lr > 0.f ? g.W : nullptr, g.lr, g.M, g.N, b.tiles_n, b.tiles_m * b.tiles_n, b.splits, g.accumulate};
#define BNS_TN(MB_, NB_) if (b.mb == MB_ && b.nb == NB_) launch_tn<MB_, NB_>(a, r, s)
  BNS_TN(128, 128); BNS_TN(128, 96); BNS_TN(128, 64); BNS_TN(128, 32);
  BNS_TN(64, 128); BNS_TN(64, 96); BNS_TN(64, 64); BNS_TN(64, 32);
#undef BNS_TN
  return hipGetLastError();
}

}  // namespace bns
