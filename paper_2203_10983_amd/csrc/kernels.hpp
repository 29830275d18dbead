// Host-side launchers of the gfx950 kernels.  Every launcher enqueues on `s` and returns the
// launch status; none synchronises.  Pointers are device pointers unless named *_host.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bns {

constexpr int kScanTile = 2048;  // elements per block in the scan / compaction kernels
inline int scan_tiles(int64_t n) { return (int)((n + kScanTile - 1) / kScanTile); }

// ---- scan.hip -------------------------------------------------------------------------------
// out[i] = add_base + sum_{j<i} in[j] for i in 0..n (n+1 entries written).  n = *n_dev if n_dev
// is non-null (n <= n_max), else n_max.  tile_sums: scratch int32[scan_tiles(n_max)+1].
// total_out (nullable): receives sum of all n inputs.
hipError_t scan_exclusive_i32(const int32_t *in, int32_t *out, int64_t n_max, const int32_t *n_dev,
                              int32_t *tile_sums, int32_t *total_out, int32_t add_base,
                              hipStream_t s);

// ---- packed weights (gemm.hip, pack_device.hpp) ------------------------------------------------
// A weight matrix laid out for the products of Eq. 2 and its backward: operand fragments in the order they are read.  split: W [N, K],
// transposed and cut into bf16 pieces, for gemm_rows (packed_bytes(K, N)); else W [K, N] for gemm_rows_f32
// (packed_bytes_f32(K, N)).  out is 16-byte aligned.
struct PackJob {
  const float *W;
  void *out;
  int32_t K, N;
  bool split, fwd;
};
constexpr int kMaxPackJobs = 16;
struct PackJobs {
  PackJob j[kMaxPackJobs];
  int32_t n = 0, units = 0;  // jobs; wavefronts' worth of work in them
};
__host__ __device__ inline int32_t pack_units(const PackJob &j) {
  return ((j.K + 31) / 32) * (j.split ? (j.N + 15) / 16 : (j.N + 31) / 32);
}
size_t packed_bytes(int32_t K, int32_t N);
size_t packed_bytes_f32(int32_t K, int32_t N);
hipError_t pack_weights(const PackJobs &jobs, hipStream_t s);

// ---- sample.hip (Algorithm 1, selection step) -------------------------------------------------
// ballots: scratch uint64[ceil(B/64)]; tile_sums: scratch int32[2 * scan_tiles(B) + 1] (half of it
// without kept_start).  epoch_dev (nullable): the epoch index is read from device memory instead of
// `epoch`.  halo_ptr + kept_start (both nullable): kept_start[r] = first + the summed lengths
// halo_ptr[b+1] - halo_ptr[b] of the kept nodes before the r-th one, r = 0..n_kept (int32[B+1]): the
// row starts of the kept nodes in the transposed subgraph, which build_subgraph reads.
// rec (nullable): rec[r] = (kept_ids[r], s_halo * dis_halo[kept_ids[r]]), as halo_records writes it.
// pack (nullable): weights to pack in the same launch, on workgroups of their own.
// count (nullable): flags and per-tile numbers of the kept boundary entries, for build_subgraph, also on workgroups of
// their own.
struct BdCount {
  int64_t e_bd = 0;
  const int32_t *bd_b = nullptr;  // boundary node of every boundary entry
  uint64_t *mask = nullptr;       // uint64[ceil(e_bd/64)]: keep flags
  int32_t *sums = nullptr;        // int32[scan_tiles(e_bd)]: kept entries per tile
  int32_t *before = nullptr;      // int32[ceil(e_bd/64)]: kept entries of the tile before the flags of a word
};
hipError_t sample_boundary(const int64_t *halo_gid, int32_t n_halo, uint64_t seed, uint32_t epoch,
                           const uint32_t *epoch_dev, uint32_t part_id, uint64_t threshold, uint64_t *ballots,
                           int32_t *tile_sums, int32_t *kept_ids, int32_t *remap, int32_t *n_kept,
                           const int32_t *halo_ptr, int32_t first, int32_t *kept_start, int2 *rec, const float *dis_halo, float s_halo,
                           const PackJobs *pack, const BdCount *count, hipStream_t s);

// ---- build_csr.hip (Algorithm 1, subgraph step) -----------------------------------------------
struct StaticSplit {       // inner / boundary split of the static CSR, built once
  int32_t *n_inner;        // int32[n_in]       inner entries in row v (scratch of set-up)
  int32_t *inner_ptr;      // int32[n_in+1]     inner entries before row v
  int32_t *bd_ptr;         // int32[n_in+1]     boundary entries before row v
  int32_t *in_col;         // int32[e_in]       inner entries, row-major
  int32_t *in_bdp;         // int32[e_in]       bd_ptr of their rows (boundary entries before the row)
  int32_t *bd_b;           // int32[e_bd]       boundary entries (boundary id), row-major
  int32_t *bd_row;         // int32[e_bd]       their rows
};
hipError_t build_static_split(int32_t n_in, const int32_t *row_ptr0, const int32_t *col0,
                              const StaticSplit &sp, int32_t *tile_sums, hipStream_t s);
// w[j] = of[col[j]]
hipError_t entry_weights(int64_t n, const int32_t *col, const float *of, float *w, hipStream_t s);
hipError_t degree_rsqrt(const int32_t *deg, int32_t n, float *dis, hipStream_t s);

// Subgraph step: the sampled CSR and the rows of the kept boundary nodes in its transpose.
struct SubgraphBuild {
  int32_t n_in, n_halo;
  int64_t e_in;
  StaticSplit sp;
  BdCount bd;
  const uint64_t *ballots;     // the keep bits written by sample_boundary (bit b%64 of word b/64)
  const int32_t *remap, *kept_ids, *n_kept;
  const int32_t *kept_start;   // row starts of the kept nodes as sample_boundary left them, int32[n_kept+1]
  const int32_t *t_in_ptr, *t_in_col, *halo_ptr, *halo_col;
  int32_t *row_ptr, *col_idx, *nnz, *t_row_ptr, *t_col_idx;
  bool static_rows;            // also write the rows of the inner nodes (the transposed inner-inner block, the same every
                               // epoch: a destination that already holds them can skip it)
};
// counted: the launch of sample_boundary has filled bd.mask and bd.sums.
hipError_t build_subgraph(const SubgraphBuild &g, bool counted, hipStream_t s);
hipError_t copy_static_rows(int32_t n_in, int64_t e_in, const int32_t *t_in_ptr, const int32_t *t_in_col,
                            int32_t *t_row_ptr, int32_t *t_col_idx, hipStream_t s);

// ---- small.hip: selection step + subgraph step of a small partition in one launch -------------
// One workgroup runs the stages of sample_boundary and build_subgraph back to back and writes the same arrays (t_row_ptr / t_col_idx must already
// hold the static rows of the inner nodes).  Its LDS holds so many boundary nodes and entries:
constexpr int kSmallMaxHalo = 8192;             // boundary nodes
constexpr int kSmallMaxBoundaryEntries = 8192;  // entries with a boundary column
// and it pays where one workgroup takes less time than the three launches of the general path, up to kSmallMaxWork (steps of 64-16-8, general and one launch, us: 600 rows with 2992 inner entries
// beside 300 boundary nodes and 7637 entries at p = 0.1, work 5452, 32.7 / 28.8; 2535 with 22045 beside 604 and 1445, 30986, 38.5 / 35.3; 1622 with
// 33052 beside 315 and 402 at p = 1, 42013, 36.5 / 34.3; 2781 with 26611 beside 1421 and 3336 at p = 0.5, 44907, 42.9 / 42.4; beyond it 8000 with 23998 beside
// 5000 and 7999 at p = 0.1, 58998, 48.7 / 53.0; 2434 with 26870 beside 2475 and 2771 at p = 1, 66347, 45.0 / 49.1; 2000 with 61556 beside
// 300 and 1397, 68216, 38.0 / 39.0; 1500 with 31262 beside 3500 and 8095 at p = 1, 81262, 42.8 / 52.3).
constexpr int kSmallMaxWork = 51200;  // inner entries + 3 per inner node + 1 per boundary node + 12 per boundary node to be expected
bool sample_build_small_fits(int32_t n_in, int32_t n_halo, int64_t e_in, int64_t e_bd, int32_t expected_kept);
// (kSmallThreads threads of a workgroup)
struct SmallArgs {
  // selection step
  const int64_t *halo_gid;
  int32_t n_halo;
  uint32_t k0, k1, epoch;
  const uint32_t *epoch_dev;
  uint32_t part_id;
  uint64_t threshold;
  uint64_t *ballots;
  int32_t *kept_ids, *remap, *n_kept, *kept_start;
  // subgraph step
  int32_t n_in, e_in, e_bd;
  StaticSplit sp;
  int32_t *row_ptr, *col_idx, *nnz;
  // transposed rows of the kept nodes
  const int32_t *halo_ptr, *halo_col;
  int32_t *t_tail_ptr, *t_col_idx;
  int2 *rec;  // per kept node: boundary index, weight
  const float *dis_halo;
  float s_halo;
};
hipError_t sample_build_small(const SmallArgs &a, const PackJobs &pack, hipStream_t s);

struct Dropout;  // defined with the GEMMs below

// ---- spmm.hip (Eq. 1 in the sampled form of Appendix A, and its transpose) ---------------------
constexpr int kSegLen = 256;  // a wavefront aggregates at most this many neighbours
// Static cut of the rows of a CSR pattern into segments of <= kSegLen entries (by the static row
// lengths; a sampled row is never longer).  Upper bounds for sizing, given rows and entries:
//   segments <= rows + nnz/kSegLen, partial slots <= 2*nnz/kSegLen, multi-segment rows <= nnz/kSegLen
struct SegPlan {
  int32_t *seg_ptr;   // int32[n_rows+1] first segment of each row
  int2 *seg_unit;     // int2[n_seg]     row of each segment and its partial-sum slot (-1: the row's only segment)
  int32_t *part_ptr;  // int32[n_rows+1] first partial-sum slot of each multi-segment row
  int32_t *mrow;      // int32[n_multi]  rows with more than one segment
  int2 *part_unit;    // int2[n_part]    row of each partial-sum slot, slot (set-up: what order is made from)
  int32_t *arrived;   // int32[4 * n_part] per row and slice, at 4 * part_ptr[row] + slice: segments finished in the launch that runs (zero between launches).  Eight slices
                      // at most, and a row that is counted has two slots at least
  int2 *order;        // int2[n_seg]     the units as launches take them: the n_part of long rows by column, then the other rows
  int32_t n_seg, n_part, n_multi;  // host copies of the totals
  int32_t max_seg;                 // segments of the longest row
  int32_t avg_len;                 // entries per row of the static pattern (launch heuristics)
};
inline int64_t seg_max_segments(int64_t rows, int64_t nnz) { return rows + nnz / kSegLen + 1; }
inline int64_t seg_max_parts(int64_t nnz) { return 2 * (nnz / kSegLen) + 2; }
inline int64_t seg_max_multi(int64_t nnz) { return nnz / kSegLen + 1; }
// Fills *plan (its arrays must be allocated to the bounds above).  Waits for the stream before the totals are read; `order` and the use of counts
// and tile_sums are complete in stream order only, after the call returns.
// tmp_a: scratch int32[n_rows], tmp_b: scratch int32[n_rows+1], counts: scratch int32[seg_max_parts(nnz)].  nnz: entries of the
// pattern, col: their columns, below n_cols.
hipError_t build_seg_plan(int32_t n_rows, int64_t nnz, const int32_t *row_ptr, const int32_t *col, int64_t n_cols, SegPlan *plan,
                          int32_t *tmp_a, int32_t *tmp_b, int32_t *counts, int32_t *tile_sums, hipStream_t s);

// A[v,:] = row_scale[v] * ( init[v,:] + sum_{u<n_in in row v} w_u H_in[u,:] + sum_{kept r in row v} Hu[r,:] )
// w_in (one weight per entry of the static inner list, which starts at w_ptr[v] for row v) / row_scale nullable (= 1).
// GCN layer: both hold d~^-1/2; mean aggregator: w_in = null,
// row_scale = 1/degree, skip_self.  plan: segmentation of the static local CSR; partials: scratch
// f32[plan.n_part * d].  part (all optional) restricts every row to entries [skip, skip+take) of
// its list, adds the initial row vector, or skips the stored self-loop.
struct SpmmRowPart {
  const int32_t *row_skip = nullptr;
  const int32_t *row_take = nullptr;
  const float *init = nullptr;
  bool skip_self = false;
  // halo_rec (from halo_records): Hu is then the whole boundary-feature table [n_halo, d] as the
  // caller holds it; kept node r reads its row halo_rec[r].x with weight as_float(halo_rec[r].y)
  const int2 *halo_rec = nullptr;
};
// rec[r] = (kept_ids[r], s_halo * dis_halo[kept_ids[r]]) for r < *n_kept (dis_halo nullable = 1): what the
// aggregate needs to read the kept boundary rows where they are instead of a gathered, scaled copy.
// pack: weights to pack in the same launch.
hipError_t halo_records(const int32_t *kept_ids, const int32_t *n_kept, int32_t n_halo, const float *dis_halo,
                        float s_halo, int2 *rec, const PackJobs &pack, hipStream_t s);
hipError_t spmm_fwd(const SegPlan &plan, int32_t n_in, int32_t d, const int32_t *row_ptr,
                    const int32_t *col_idx, const float *w_in, const int32_t *w_ptr, const float *row_scale,
                    const float *H_in, const float *Hu, float *partials, float *A,
                    const SpmmRowPart &part, bool long_rows_only, bool relu, hipStream_t s,
                    int32_t d_store = 0);
// d_store (spmm_fwd and spmm_bwd; 0 = d): the sources and partial sums have rows of d floats of which
// only the first d_store count (rows padded to a multiple of 4 floats so that a narrow odd width is
// gathered with 16-byte loads); the outputs are dense [., d_store].  Then d < 128, no mask, no init.
// pad_rows makes such a padded copy (pad columns zero).  long_rows_only: the partial sums of the rows of several segments, for spmm_gemm_fwd,
// and nothing else.
hipError_t pad_rows(int32_t n_rows, int32_t d, int32_t ld, const float *src, float *dst, hipStream_t s);
// Aggregate and update of one GCN layer in one kernel (Eq. 1 then Eq. 2): a workgroup aggregates 64
// rows into LDS (and stores them to A, which the backward pass needs), then multiplies the tile by
// W on the matrix cores while other workgroups of the same compute unit keep gathering.  The partial sums of
// rows cut into several segments must have been left in `partials` by spmm_fwd(..., long_rows_only = true).
// Needs d_in % 4 == 0 and 64 < d_in <= 128 (spmm_gemm_fwd_supported).
// concat_self: the update of the mean-aggregator layer, H_out = act([A | H_in] W) with W [2 d_in, d_out]
// (neighbour half first): the tile is multiplied by W_n, overwritten with the rows' own features and
// multiplied by W_s into the same accumulators; needs d_out <= 256 (spmm_gemm_fwd_concat_supported).
bool spmm_gemm_fwd_supported(int32_t d_in);
bool spmm_gemm_fwd_concat_supported(int32_t d_in, int32_t d_out);
hipError_t spmm_gemm_fwd(const SegPlan &plan, int32_t n_in, int32_t d_in, int32_t d_out, const int32_t *row_ptr,
                         const int32_t *col_idx, const float *w_in, const int32_t *w_ptr, const float *row_scale,
                         const float *H_in, const float *Hu, float *partials, float *A,
                         const SpmmRowPart &part, const float *W, float *H_out, bool relu,
                         const Dropout &drop, hipStream_t s, bool concat_self = false);
// For stacked column u < n_in + *n_kept:  g = sum_{v in t_row u} w_v dA[v,:];
//   u <  n_in: dH_in[u,:] = row_scale[u] * (init[u,:] + g)  (zeroed where mask_src[u,:] <= 0 if given)
//   u >= n_in: dhalo[u-n_in,:] = s_halo * dis_halo[kept_ids[u-n_in]] * g   (skipped if dhalo null)
// Weights per entry: w_in in the order of the transposed inner-inner block, w_halo in that of the boundary nodes' static
// lists (halo_ptr).  avg_len: entries to be expected per row of the launch, expected_halo: about *n_kept (any number is walked).  row_scale, dis_halo, init nullable.  plan: segmentation of the transposed inner-inner block.
hipError_t spmm_bwd(const SegPlan &plan, int32_t n_in, int32_t n_halo, int32_t d,
                    const int32_t *t_row_ptr, const int32_t *t_col_idx, const int32_t *kept_ids,
                    const int32_t *n_kept, const float *w_in, const float *w_halo, const int32_t *halo_ptr, const float *row_scale,
                    const float *dis_halo, float s_halo, const float *dA, const float *mask_src,
                    const float *init, bool skip_self, int32_t avg_len, float *partials, float *dH_in, float *dhalo,
                    int32_t expected_halo, hipStream_t s, int32_t d_store = 0);

// ---- gemm_f32.hip (Eq. 2; fp32 MFMA), gemm.hip (its backward; fp32 on the bf16 MFMA) -------------
// Dropout on a hidden layer's output (training set-up of Section 4): element (row, col) is kept iff
// the first word of Philox-4x32-10 on the counter (row, col, c2, epoch) under key (k0, k1) is below
// `threshold`; kept elements are multiplied by `scale` = 1/(1-q).  scale == 0: no dropout.
struct Dropout {
  uint64_t threshold = 0;
  float scale = 0.f;
  uint32_t k0 = 0, k1 = 0, c2 = 0, epoch = 0;
  const uint32_t *epoch_dev = nullptr;  // nullable: the epoch index is read from device memory
};
// ---- tile.hip: aggregate and update of a layer of a small partition in one launch --------------
// As spmm_fwd and then gemm_rows_f32 on [A | H_in (sage)] W with the plain W: the same bits.  concat: the two halves of the mean
// aggregator's update are one product (else two, added).  Neither A nor H_out may share memory with H_in, Hu or W.
// loss (nullable, d_out <= kTileLossWidth, no relu): of the output, as loss_softmax_ce, in the same launch.
struct TileLoss {
  const int32_t *labels = nullptr;
  float *dZ = nullptr, *dZ_pad = nullptr, *partials = nullptr;
  int32_t ld = 0, n_partials = 0;  // n_partials: set by the call
};
constexpr int kTileLossWidth = 128;
bool tile_layer_supported(const SegPlan &plan, int32_t d_in, int32_t d_out);
hipError_t tile_layer_fwd(const SegPlan &plan, int32_t n_in, int32_t d_in, int32_t d_out, const int32_t *row_ptr,
                          const int32_t *col_idx, const float *w_in, const int32_t *w_ptr, const float *row_scale,
                          const float *H_in, const float *Hu, float *partials, float *A, const SpmmRowPart &part, const float *W,
                          float *H_out, bool relu, const Dropout &drop, bool sage, bool concat, TileLoss *loss, hipStream_t s);

// dH[u,:] = alpha * (P^T dZ [+ dZ of u (sage: by the second half of W)]) W^T, zeroed where mask <= 0 (nullable), and for the kept
// boundary nodes (dhalo nullable) without alpha and mask: as spmm_bwd (its arguments; dZ has rows of d floats, zeros from d_out
// on) and gemm_rows (on W packed as one matrix), the aggregate first.  Neither dH nor dhalo may share memory with dZ, W or mask.
bool tile_layer_bwd_supported(int32_t d, int32_t d_in, bool sage);
hipError_t tile_layer_bwd(const SegPlan &plan, int32_t n_in, int32_t n_halo, int32_t d, int32_t d_in, int32_t d_out, const int32_t *t_row_ptr,
                          const int32_t *t_col_idx, const int32_t *kept_ids, const int32_t *n_kept, const float *w_in, const float *w_halo,
                          const int32_t *halo_ptr, const float *row_scale, const float *dis_halo, float s_halo, const float *dZ,
                          const float *W, const void *Bp, const float *mask, float alpha, bool sage, float *partials, float *dH, float *dhalo,
                          int32_t expected_halo, hipStream_t s);

// ---- first.hip: sample_build_small and the first layer's tile_layer_fwd in one launch ------------
// For a plan without rows of several segments and a layer that is not the last.  cached (nullable): the sum over the inner entries, as
// SpmmRowPart::init.  Same bits as the two launches.
hipError_t sample_build_first(const SmallArgs &small, const PackJobs &pack, int32_t d_in, int32_t d_out, const float *w_in, const float *row_scale,
                              const float *H_in, const float *halo_h, float *A, const float *cached, const float *W, float *H_out,
                              bool relu, const Dropout &drop, bool sage, bool concat, const SegPlan &plan, hipStream_t s);

// C[M,N] = [A | A2] B (+ the previous C if accumulate), B [K,N] packed; then, if relu, max(., 0) and dropout (when
// drop.scale != 0).  A, A2 [M, lda]: the depth below a_split (a multiple of 16) is A's, the rest A2's (nullable).
// pad: the columns N..ldc-1 are set to zero (ldc at most N rounded up to a multiple of 4; not with relu or
// accumulate).
// rec (nullable; from halo_records): in the same launch C_rec[r] = as_float(rec[r].y) * A_rec[rec[r].x] B for r < *m2_dev
// (<= M2, about m2_expected, which shapes the launch); not with A2, relu or accumulate.
struct RowsF32 {
  int32_t M, N, K;
  const float *A, *A2;
  int32_t lda, a_split;
  const void *Bp;
  float *C;
  int32_t ldc;
  bool relu, pad, accumulate;
  const int2 *rec;
  const float *A_rec;
  float *C_rec;
  int32_t M2, m2_expected;
  const int32_t *m2_dev;
  Dropout drop;
};
hipError_t gemm_rows_f32(const RowsF32 &g, hipStream_t s);
// The same from W [K, N] by the split products of gemm.hip (Bp packed accordingly).
hipError_t gemm_fwd_split(const RowsF32 &g, const float *W, hipStream_t s);

// C[M,N] = alpha * A B with A [M,K], B [K,N] packed and split, from W [N,K].  At most one of: C2 (nullable): columns from c_split (a
// multiple of 4) on go to C2, both with row stride ldc; mask (nullable, [M, ldc]): C is zeroed where mask <= 0.
// A_more (nullable): in the same launch C_more[r] = A_more[r] B for r < *m2_dev (<= M2, about m2_expected); not with C2.
// A2 (nullable, [M, K]; not with C2): C = alpha * (A B + A2 B2), B2 packed behind B, from the [N, K] that follow in W.
struct RowsGemm {
  int32_t M, N, K;
  const float *A, *W;
  const void *Bp;
  float *C, *C2;
  int32_t ldc, c_split;
  float alpha;
  const float *mask;
  const float *A_more;
  float *C_more;
  int32_t M2, m2_expected;
  const int32_t *m2_dev;
  // rows of A are lda apart (fwd unset: K)
  int32_t lda;
  // a forward product, W [K, N]: its arguments as in RowsF32 (A_rec is A_more)
  bool fwd;
  const float *A2;
  int32_t a_split;
  bool relu, pad, accumulate;
  const int2 *rec;
  Dropout drop;
};
hipError_t gemm_rows(const RowsGemm &g, hipStream_t s);

// inv[i] = deg[i] > 1 ? 1 / (deg[i] - 1) : 0   (deg counts the self-loop)
hipError_t degree_inverse(const int32_t *deg, int32_t n, float *inv, hipStream_t s);

// C[M,N] = [A | A2]^T B with B [K,N] and A [K, M], or A, A2 [K, a_split] and [K, M - a_split] (both with row
// stride a_split, M = 2 a_split); accumulate: adds to the C of the job before it instead (same M, N).  The depth is split
// over the chip and summed in a fixed order; partials: scratch of
// gemm_tn_partials(M, N, K, depth of the other part of the same gradient or 0) floats per job.  rows
// (nullable, [K]): the rows of A are those.  k_dev (nullable): depth on the device, *k_dev <= K and about k_expected.  lr > 0: also
// W -= lr * C, the plain update of Algorithm 1.  A batch of up to kMaxTnJobs jobs shares its launches; in the last of
// them *loss.out (nullable) becomes the sum of loss.n partial losses.
struct TnGemm {
  int32_t M, N, K;
  const float *A, *A2, *B;
  int32_t a_split;
  const int32_t *rows;
  float *C, *partials;
  bool accumulate;
  const int32_t *k_dev;
  int32_t k_expected;
  float *W;
  float lr;
};
struct TnLoss {
  const float *partials = nullptr;
  int32_t n = 0;
  float *out = nullptr;
  uint32_t *bump = nullptr;  // nullable, with out: *bump += 1 (the epoch of a captured step, whose last launch this is)
};
// Do a and b, of na and nb floats, share memory?
inline bool overlap(const float *a, size_t na, const float *b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb * sizeof(float) && y < x + na * sizeof(float);
}
constexpr int kMaxTnJobs = 16;
size_t gemm_tn_partials(int32_t M, int32_t N, int32_t K, int32_t K_other);
hipError_t gemm_tn(const TnGemm *g, int32_t n, const TnLoss &loss, hipStream_t s);

// ---- loss.hip (Algorithm 1, loss step) ---------------------------------------------------------
constexpr int kLossBlocks = 8192;  // partials: scratch f32[kLossBlocks]
// Leave *n_partials partial losses, which gemm_tn adds up.  dZ_pad (nullable): the gradient once more in rows padded by
// zeros to ld floats (as pad_rows makes them; ld < C + 4).
hipError_t loss_softmax_ce(int32_t n, int32_t C, const float *logits, const int32_t *labels,
                           float *dZ, int32_t ld, float *dZ_pad, float *partials, int32_t *n_partials, hipStream_t s);
hipError_t loss_sigmoid_bce(int32_t n, int32_t C, const float *logits, const uint8_t *labels,
                            float *dZ, int32_t ld, float *dZ_pad, float *partials, int32_t *n_partials, hipStream_t s);
// Dropout applied in place to H[n_rows, d] (for layers whose ReLU sits in the aggregate's store).
hipError_t dropout_inplace(int32_t n_rows, int32_t d, float *H, const Dropout &drop, hipStream_t s);
// out = scale * dH where H > 0 else 0 (H, out [n_rows, d] nullable: dH as it is).  pad (nullable): the result once more in rows padded by
// zeros to ld floats, a multiple of 4.  pack: weights to pack in the same launch.
hipError_t relu_mask(int32_t n_rows, int32_t d, const float *dH, const float *H, float scale, float *out, int32_t ld, float *pad,
                     const PackJobs &pack, hipStream_t s);
// W -= lr * dW on n weights, as gemm_tn does it on the way (same bits): for a step whose update is timed by itself.
hipError_t sgd_update(int64_t n, float *W, const float *dW, float lr, hipStream_t s);
// Adam step t (1-based) on n weights; m, v are the caller's moment buffers.
hipError_t adam_update(int64_t n, float *W, const float *dW, float *m, float *v, float lr, float b1,
                       float b2, float eps, int32_t t, hipStream_t s);
// *counter = value (one thread; the device-side epoch index of graph replay)
hipError_t set_counter(uint32_t *counter, uint32_t value, hipStream_t s);

}  // namespace bns
