// A layer of a small partition in one launch, forward: aggregate (Eq. 1), then update (Eq. 2) of a few rows in one workgroup; and
// backward: transposed aggregate, then product with W^T.
//
// On some thousand rows neither step fills the chip: a launch is 2 to 3 us of starting and draining beside about 2 us of
// dependent reads, whatever its size.  A workgroup of 8 wavefronts owns a tile of 8 or 16 rows, gathers them into LDS with the
// code and the order of sums of spmm_kernel, and multiplies them by W with v_mfma_f32_16x16x4_f32, a wavefront per 16 or
// 32 columns.  That instruction is a chain of fused multiply-adds in depth order, as v_mfma_f32_32x32x2_f32 is (40960 sums of 128 products of
// operands of any size: equal bits, and equal to fmaf), so that the results are those of spmm_kernel and gemm_rows_f32_kernel.
// The last layer forms the softmax loss and its gradient on the way (steps of 500 rows 64-16-8 36 -> 34 us, 3500 rows
// 64-128-47 3 % less; the sigmoid loss, an exponential and a logarithm per element of few columns, gained nothing here).
// W is asked for before the gather, straight from the caller's matrix: 16 columns of 4 depths are a load of 256 bytes.
#include "tile_device.hpp"

namespace bns {

namespace {

template <int LPR, int VW, bool SAGE, bool LOSS = false>
__global__ void __launch_bounds__(kTileWaves * kWave, 4) tile_layer_kernel(const TileArgs f) {
  __shared__ __attribute__((aligned(16))) float As[SAGE ? 2 : 1][kTileRows * kTileLd];
  tile_layer<LPR, VW, SAGE, LOSS>(f, blockIdx.x, threadIdx.x, As, [&](int row0, int rows, auto put) { gather_tile<LPR>(f.sp, row0, rows, put); });
}

// The gradient of the layer's input: dH = mask(P^T dZ W^T), the rows of the inner nodes and, on the workgroups behind theirs,
// those of the kept boundary nodes.  The transposed aggregate comes first whatever the widths: its rows stay in LDS.  The product is
// that of gemm_rows_kernel, on the same packed weights (of a chain of fp32 instructions the error was 1.1 to 1.9 times that of the split).
struct TileBwdArgs {
  SpmmArgs sp;          // src0: dZ with rows of d floats, of which d_out count (the others are zero); out_scale0, s_halo, ...
  const float *W;       // [d_in, d_out]; SAGE: [2 d_in, d_out]
  const void *Bp;       // the same, packed and split
  const float *mask;    // nullable: [n_in, d_in]
  float *dH, *dhalo;    // [n_in, d_in], [.., d_in]
  int32_t d_in, d_out, rows, n_tiles;  // tiles of inner rows
  float alpha;          // of the inner rows
};

template <int LPR, bool SAGE>
__global__ void __launch_bounds__(kTileWaves * kWave, 4) tile_layer_bwd_kernel(const TileBwdArgs f) {
  using V = typename Vec<4>::T;
  constexpr int S = (LPR * 4 + 31) / 32;  // depth steps at most
  __shared__ __attribute__((aligned(16))) float As[SAGE ? 2 : 1][kTileRows * kTileLd];
  const SpmmArgs &a = f.sp;
  const int lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int d = a.d, nvec = d / 4, N = f.d_in, K = f.d_out, steps = (K + 31) / 32;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int n0 = wid * 16;  // the wavefront's columns; a lane ends up with n0 + 4 (lane / 16) .. + 3 of row lane % 16
  const int T = ((SAGE ? 2 * N : N) + 15) / 16;
  // Column `from` + n0 + lane % 16 of the packed weights (N % 4 == 0 where `from` is not 0), zeros behind the last one.  Those of the
  // first step are asked for before the gather, the others behind it: more of them before it hold up its first reads (step of
  // 64-100-100-47, mean aggregator, 1500 rows: 79.1 us, with two 80.8, four 81.7).
  auto load_w = [&](bf16x8 (&w)[S][3], int from, int s0, int s1) {
    if (n0 >= N) return;
    const int col = min(from + n0 + l16, T * 16 - 1);
    const char *p = static_cast<const char *>(f.Bp) + (size_t)(col / 16) * kFragSet + (g4 * 16 + col % 16) * 16;
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (s >= s0 && s < s1 && s < steps)
#pragma unroll
        for (int i = 0; i < 3; ++i) w[s][i] = *reinterpret_cast<const bf16x8 *>(p + (size_t)s * T * kFragSet + i * kFragBytes);
  };
  const int n_kept = a.n_extra_dev ? scalar_load(a.n_extra_dev, 0) : 0;
  const bool halo = (int)blockIdx.x >= f.n_tiles;
  for (int tile = halo ? (int)blockIdx.x - f.n_tiles : (int)blockIdx.x;; tile += (int)gridDim.x - f.n_tiles) {
    const int r0 = tile * f.rows;  // of the inner or of the kept boundary rows
    if (r0 >= (halo ? n_kept : a.n_split)) return;
    const int rows = min(f.rows, (halo ? n_kept : a.n_split) - r0), row0 = halo ? a.n_split + r0 : r0;
    bf16x8 w[S][3];
    load_w(w, 0, 0, 1);
    const bool own = SAGE && !halo;
    const int pad = 8 * steps - nvec;  // pieces behind a row up to the depth of the product
    for (int idx = threadIdx.x; idx < kTileRows * pad; idx += kTileWaves * kWave)
#pragma unroll
      for (int t = 0; t < (SAGE ? 2 : 1); ++t)
        *reinterpret_cast<V *>(&As[t][idx / pad * kTileLd + (nvec + idx % pad) * 4]) = V{0.f, 0.f, 0.f, 0.f};
    if (own)
      for (int idx = threadIdx.x; idx < rows * nvec; idx += kTileWaves * kWave) {
        const int r = idx / nvec, c4 = idx - r * nvec;
        *reinterpret_cast<V *>(&As[SAGE ? 1 : 0][r * kTileLd + c4 * 4]) = reinterpret_cast<const V *>(a.src0 + (size_t)(row0 + r) * d)[c4];
      }
    const int col = n0 + 4 * g4, left = N - col;
    const bool stores = l16 < rows && left > 0;
    const size_t at = (size_t)(r0 + l16) * N + col;
    f32x4 mask = {1.f, 1.f, 1.f, 1.f};
    if (f.mask && !halo && stores) {
      if (left >= 4) mask = *reinterpret_cast<const f32x4u *>(f.mask + at);
      else
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (e < left) mask[e] = f.mask[at + e];
    }
    gather_tile<LPR>(a, row0, rows, [&](int row, int piece, const float (&acc)[1][4]) {
      float scale = 1.f;
      if (!halo) {
        if (a.out_scale0) scale = scalar_load(a.out_scale0, row);
      } else {
        scale = a.dis_halo ? a.s_halo * scalar_load(a.dis_halo, scalar_load(a.kept_ids, row - a.n_split)) : a.s_halo;
      }
      if (piece < nvec) *reinterpret_cast<V *>(&As[0][(row - row0) * kTileLd + piece * 4]) = V{acc[0][0], acc[0][1], acc[0][2], acc[0][3]} * scale;
    });
    load_w(w, 0, 1, S);
    __syncthreads();
    if (n0 < N) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      auto product = [&](const float *tile_rows, int from) {
        const float *as = tile_rows + l16 * kTileLd + 4 * g4;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (s < steps) {
            const Frag3 fa[1] = {split8(*reinterpret_cast<const f32x4 *>(as + 32 * s), *reinterpret_cast<const f32x4 *>(as + 32 * s + 16))};
            const Frag3 fb = {{w[s][0], w[s][1], w[s][2]}};
            f32x4 part[1];
            mfma_split<1>(part, fb, fa);
            sum += part[0];
            if (from == 0 && own) load_w(w, N, s, s + 1);  // the other half's
          }
        v += (from + col) / 16 & 1 ? -sum : sum;  // odd tiles are packed negated
      };
      product(As[0], 0);
      if (own) {
        product(As[SAGE ? 1 : 0], N);
      }
      if (stores && nonfinite_seed(0.f, v) != 0.f) {  // (NaN)
#pragma unroll 1
        for (int e = 0; e < 4; ++e) {
          if (e < left && !is_finite(v[0])) {
            float x = 0.f;
#pragma unroll 1
            for (int h = 0; h < (own ? 2 : 1); ++h)
#pragma unroll 1
              for (int k = 0; k < K; ++k) x = fmaf(As[SAGE ? h : 0][l16 * kTileLd + k], f.W[((size_t)h * N + col + e) * K + k], x);
            v[0] = x;
          }
          v = f32x4{v[1], v[2], v[3], v[0]};
        }
      }
      if (stores) {
        if (!halo)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = f.mask ? mask[e] > 0.f ? v[e] * f.alpha : 0.f : v[e] * f.alpha;
        float *const to = (halo ? f.dhalo : f.dH) + at;
        if (left >= 4) *reinterpret_cast<f32x4u *>(to) = v;
        else
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (e < left) to[e] = v[e];
      }
    }
    if (!halo) return;
    __syncthreads();  // the tile is read before it is filled again
  }
}

}  // namespace

bool tile_layer_supported(const SegPlan &plan, int32_t d_in, int32_t d_out) {
  // rows of 4 to 32 lanes (128 floats are cut into slices from 64 entries a row on); the weights of 32 columns at 128
  // depths are more registers than there are
  return d_in % 4 == 0 && d_in > 8 && d_in <= kTileDepth && (d_in < kTileDepth || plan.avg_len < 64) && d_out >= 1 &&
         d_out <= (d_in <= 64 ? 32 : 16) * kTileWaves;
}

hipError_t tile_layer_fwd(const SegPlan &plan, int32_t n_in, int32_t d_in, int32_t d_out, const int32_t *row_ptr,
                          const int32_t *col_idx, const float *w_in, const int32_t *w_ptr, const float *row_scale,
                          const float *H_in, const float *Hu, float *partials, float *A, const SpmmRowPart &part, const float *W,
                          float *H_out, bool relu, const Dropout &drop, bool sage, bool concat, TileLoss *loss, hipStream_t s) {
  if (!tile_layer_supported(plan, d_in, d_out) || (loss && d_out > kTileLossWidth)) return hipErrorInvalidValue;
  if (n_in <= 0) return hipSuccess;
  TileArgs f;
  f.sp = spmm_fwd_args(plan, n_in, d_in, row_ptr, col_idx, w_in, w_ptr, row_scale, H_in, Hu, partials, A, part);
  f.W = W;
  f.H_self = sage ? H_in : nullptr;
  f.H_out = H_out;
  f.d_out = d_out;
  f.rows = tile_rows(n_in);
  f.relu = relu;
  f.concat = concat;
  f.drop = drop;
  if (loss) f.loss = *loss;
  const unsigned blocks = (unsigned)((n_in + f.rows - 1) / f.rows);
  if (loss) loss->n_partials = (int32_t)blocks;
#define BNS_TILE_KIND(LPR, VW, LOSS)                                                                  \
  do {                                                                                                \
    if (sage) tile_layer_kernel<LPR, VW, true, LOSS><<<blocks, kTileWaves * kWave, 0, s>>>(f);       \
    else tile_layer_kernel<LPR, VW, false, LOSS><<<blocks, kTileWaves * kWave, 0, s>>>(f);           \
  } while (0)
#define BNS_TILE(LPR, VW)                                     \
  do {                                                        \
    if (VW == 1 && loss) BNS_TILE_KIND(LPR, 1, true);         \
    else BNS_TILE_KIND(LPR, VW, false);                       \
  } while (0)
  const bool wide = d_out > 16 * kTileWaves;
  if (d_in > 64) BNS_TILE(32, 1);
  else if (d_in > 32) { if (wide) BNS_TILE(16, 2); else BNS_TILE(16, 1); }
  else if (d_in > 16) { if (wide) BNS_TILE(8, 2); else BNS_TILE(8, 1); }
  else { if (wide) BNS_TILE(4, 2); else BNS_TILE(4, 1); }
#undef BNS_TILE
#undef BNS_TILE_KIND
  return hipGetLastError();
}

bool tile_layer_bwd_supported(int32_t d, int32_t d_in, bool sage) {
  return d % 4 == 0 && d > 4 && d <= kTileDepth && d_in <= 16 * kTileWaves && (!sage || d_in % 4 == 0);
}

hipError_t tile_layer_bwd(const SegPlan &plan, int32_t n_in, int32_t n_halo, int32_t d, int32_t d_in, int32_t d_out, const int32_t *t_row_ptr,
                          const int32_t *t_col_idx, const int32_t *kept_ids, const int32_t *n_kept, const float *w_in, const float *w_halo,
                          const int32_t *halo_ptr, const float *row_scale, const float *dis_halo, float s_halo, const float *dZ,
                          const float *W, const void *Bp, const float *mask, float alpha, bool sage, float *partials, float *dH, float *dhalo,
                          int32_t expected_halo, hipStream_t s) {
  if (!tile_layer_bwd_supported(d, d_in, sage) || d_out > d || d_out < 1) return hipErrorInvalidValue;
  if (n_in <= 0) return hipSuccess;
  const bool halo_rows = dhalo && n_halo > 0;
  TileBwdArgs f{};
  SpmmArgs &a = f.sp;
  a.plan = plan; a.n_extra_dev = halo_rows ? n_kept : nullptr; a.d = a.d_store = d;
  a.row_ptr = t_row_ptr; a.col_idx = t_col_idx; a.n_split = n_in;
  a.src0 = dZ; a.w_in = w_in; a.w_ptr = t_row_ptr; a.w_halo = w_halo; a.halo_ptr = halo_ptr; a.partials = partials;
  a.out_scale0 = row_scale; a.kept_ids = kept_ids; a.dis_halo = dis_halo; a.s_halo = s_halo; a.skip_self = sage;
  f.W = W;
  f.Bp = Bp;
  f.mask = mask;
  f.dH = dH;
  f.dhalo = dhalo;
  f.d_in = d_in;
  f.d_out = d_out;
  f.rows = tile_rows(n_in + (halo_rows ? expected_halo : 0));
  f.n_tiles = (n_in + f.rows - 1) / f.rows;
  f.alpha = alpha;
  // (any number of boundary rows is walked)
  const unsigned blocks = (unsigned)(f.n_tiles + (halo_rows ? expected_halo / f.rows + 1 : 0));
#define BNS_TILE(LPR)                                                                           \
  do {                                                                                          \
    if (sage) tile_layer_bwd_kernel<LPR, true><<<blocks, kTileWaves * kWave, 0, s>>>(f);       \
    else tile_layer_bwd_kernel<LPR, false><<<blocks, kTileWaves * kWave, 0, s>>>(f);           \
  } while (0)
  if (d > 64) BNS_TILE(32);
  else if (d > 32) BNS_TILE(16);
  else if (d > 16) BNS_TILE(8);
  else if (d > 8) BNS_TILE(4);
  else BNS_TILE(2);
#undef BNS_TILE
  return hipGetLastError();
}

}  // namespace bns
