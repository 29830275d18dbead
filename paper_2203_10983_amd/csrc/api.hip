// C ABI of the BNS-GCN partition step: context, workspace carving, argument checks and the
// sequencing of the kernels.  See include/bns_gcn.h for the contract of every entry point.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/bns_gcn.h"
#include "kernels.hpp"

using namespace bns;

const char *bns_noalloc_last_error();  // noalloc.hip: error text of the context-free calls on this thread

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Walks the workspace once; used both to size it and to hand out pointers.
struct Carver {
  char *base;
  size_t off = 0;
  explicit Carver(void *b) : base(static_cast<char *>(b)) {}
  template <typename T> T *take(size_t count) {
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += align_up(count * sizeof(T));
    return p;
  }
};

struct Layout {
  // static, filled at set-up
  float *dis_in, *dis_halo;
  StaticSplit split;
  // scratch shared by all calls
  int32_t *tile_sums, *kept_start;
  uint64_t *ballots;
  uint64_t *bd_mask;   // keep flags of the boundary entries, their number per tile and per tile before each word
  int32_t *bd_sums, *bd_before;
  // boundary rows at the output width: Hu of GCN layers that shrink and of mean-aggregator layers that gather first (their gradient), Hu2 of update-first layers
  float *Hu, *Hu2, *G0, *G1, *G2, *loss_partials;
  int2 *halo_rec;  // per kept boundary node: (boundary index, weight) for the aggregates that read the rows in place
  // weight of every static entry with an inner column: forward (GCN only), transposed inner block, boundary nodes' lists
  float *w_fwd, *w_bwd, *w_halo;
  float *inv_deg;            // 1 / (full-graph degree) of the inner nodes, for the mean aggregator
  SegPlan plan_f, plan_b;   // segmentation of the static CSR and of the transposed inner block
  int32_t *seg_tmp_a, *seg_tmp_b;
  float *spmm_partials;
  float *C0;                // cached inner part of layer 1's aggregate (n_in x d_0)
  // state of bns_train_step
  int32_t *kept_ids, *remap, *counters;
  int32_t *row_ptr, *col_idx, *t_row_ptr, *t_col_idx;
  std::vector<float *> A, H;  // index 1..L
  std::vector<char *> Wf, Wb;  // index 1..L: the layer's weights packed for H W and for dZ W^T
  // index 1..L: partial sums of the layer's weight gradient (of its boundary part); transposed aggregate of an
  // update-first layer's gradient, inner and boundary rows
  std::vector<float *> tn, tn2, G_in, G_halo;
  std::vector<float *> dZ;    // index 1..L: gradient w.r.t. the pre-activation of layer l (bns_train_step)
};

}  // namespace

// Optional instrumentation: HIP events around every kernel class of bns_train_step.
struct Profiler {
  uint32_t mask = 0;
  std::vector<hipEvent_t> start, stop;
  std::vector<int> phase;
  size_t used = 0;
  ~Profiler() {
    for (hipEvent_t e : start) (void)hipEventDestroy(e);
    for (hipEvent_t e : stop) (void)hipEventDestroy(e);
  }
};

struct bns_ctx {
  Profiler prof;
  bns_partition_desc part;
  std::vector<int32_t> dims;
  int32_t n_layers, loss_kind, layer_kind;
  Layout ws;
  // latest sample / subgraph the layer calls work on
  const int32_t *cur_kept = nullptr, *cur_remap = nullptr, *cur_n_kept = nullptr;
  const int32_t *cur_row_ptr = nullptr, *cur_col_idx = nullptr, *cur_t_row_ptr = nullptr,
                *cur_t_col_idx = nullptr;
  const float *cache_X = nullptr;  // features whose inner aggregate sits in ws.C0 (nullptr: none)
  double drop_q = 0.0;             // dropout rate on hidden activations (0: none)
  uint64_t cur_seed = 0;           // seed / epoch of the latest boundary sample: the dropout draw uses them
  uint32_t cur_epoch = 0;
  const uint32_t *cur_epoch_dev = nullptr;
  bool cur_counted = false;             // the kept boundary entries of the latest sample are counted in the workspace
  const int32_t *drawn = nullptr;       // remap of the sample whose keep bits and row starts sit in the workspace: the latest that ran
  bool ws_built = false;                // a subgraph has been written to the workspace arrays (a capture alone writes none)
  hipGraphExec_t graph_exec = nullptr;  // captured training step (bns_graph_capture)
  std::string err;
};

namespace {

// A GCN layer that shrinks its width by a quarter or more is run update first in bns_train_step:
// (P (H W)) instead of ((P H) W), so that the aggregate moves d_out instead of d_in floats per entry.
bool update_first_shape(int layer_kind, int d_in, int d_out) {
  return layer_kind == 0 && (int64_t)d_out * 4 <= (int64_t)d_in * 3;
}

// Row stride of an operand that is gathered at the output width d_out of a layer: a narrow width
// that is not a multiple of 4 is padded to one (the aggregate then reads 16 bytes per lane and
// several neighbours per load instruction) as long as the padded rows fit the buffers, which are
// sized for the input width.
int gather_stride(int d_in, int d_out) {
  const int ld = (d_out + 3) & ~3;
  return (d_out % 4 != 0 && ld < 128 && ld <= d_in) ? ld : d_out;
}

// Aggregate and update of a layer in one kernel?  The kernel's two phases (gather, product) do not
// overlap, so it pays only while the product is short beside the gather: measured on the five
// workloads, up to about 6.5 multiply-adds of the update per gathered feature element (GCN layers of
// workload 5: 4.4 and 6.0, faster in one kernel; mean-aggregator layers, whose update is twice as
// deep: workload 3 at 5.1 faster, workload 5 at 8.9 and 11.9 slower).
// Its workgroups own 64 rows, so that few rows leave the chip short of them, and rows of several segments need a launch
// before it.  Both sides timed, one kernel / two (us, 128 x 128): without such rows 20000 rows of 20 entries 50 / 42, 30000
// 61 / 62, 45000 88 / 90, 100000 197 / 205; with them 45000 80 / 77, 65000 115 / 106, 100000 174 / 168, 200000 314 / 317 (steps
// of 65000, 130000 and 300000 rows, hidden width 128: 385 / 372, 662 / 672, 1344 / 1391).
constexpr int kOneKernelMinRows = 32768, kOneKernelMinRowsLong = 98304;
bool one_kernel_layer(const bns_ctx *ctx, int d_in, int d_out) {
  const bns_partition_desc &part = ctx->part;
  const int layer_kind = ctx->layer_kind;
  if (part.n_in < (ctx->ws.plan_f.n_multi > 0 ? kOneKernelMinRowsLong : kOneKernelMinRows)) return false;
  if (layer_kind == 0) return spmm_gemm_fwd_supported(d_in);  // every GCN shape measured so far gains
  if (!spmm_gemm_fwd_concat_supported(d_in, d_out)) return false;
  const double avg_len = (double)part.nnz0 / (double)part.n_in;
  return 2.0 * d_out <= 6.5 * avg_len;
}

// The concatenated update [z | h] [W_n ; W_s] of the mean-aggregator layer as one product: the seam must
// not cut the 16-deep groups that a depth is zero-padded to.
bool concat_in_one(int d_in) { return d_in % 16 == 0; }

// Aggregate and update of a layer of a small partition in one launch, a few rows per workgroup?  A launch and a pass over
// the aggregate less; with more rows than fill the chip the weights, read anew for every tile, cost more than they save, and a row
// of several segments, which its workgroup gathers alone, does so sooner.  Steps, two launches per layer / one (us): without such
// rows 500 rows 64-16-8 45 / 37, 500 rows 128-128-128-47 77 / 59, 3000 rows of 10 entries 108 / 93, 6500 129 / 114, 9000 141 / 137
// and with 45 entries 162 / 164, 12000 160 / 158; with them 1000 rows of 45 entries 118 / 102, 3000 136 / 130, 4500 146 / 155.
constexpr int kTileMaxRows = 8192, kTileMaxRowsLong = 3584, kTileMaxSegments = 8;
bool tile_layer(const bns_ctx *ctx, int layer) {
  const SegPlan &plan = ctx->ws.plan_f;
  return ctx->part.n_in <= (plan.n_multi > 0 ? kTileMaxRowsLong : kTileMaxRows) && plan.max_seg <= kTileMaxSegments &&
         tile_layer_supported(plan, ctx->dims[layer - 1], ctx->dims[layer]);
}

// Its backward pass, likewise: the transposed aggregate (at the output width, in rows of gather_stride floats), then the product?  (The two
// launches multiply first where the output is not narrower and in mean-aggregator layers: the same result up to rounding.)
// rows: inner ones and expected boundary rows.  Here the two launches keep up sooner (steps, two per layer and one, us: 64-16-8
// 500 rows 38 / 36, 64-128-128-47 700 rows 61 / 57, 1500 of 15 entries 84 / 81, 2500 91 / 90, 5000 98 / 100; mean aggregator
// 64-64-128-8 1500 rows 79 / 76, 5000 107 / 107; with rows of several segments 64-128-128-47, 1500 rows of 15 entries 103 / 101, of
// 45 115 / 118).
constexpr int kTileBwdMaxRows = 3072, kTileBwdMaxSegments = 3, kTileBwdMaxLen = 32;
bool tile_layer_bwd(const bns_ctx *ctx, int layer, int64_t rows) {
  const SegPlan &plan = ctx->ws.plan_b;
  return rows <= kTileBwdMaxRows && (plan.n_multi == 0 || (plan.max_seg <= kTileBwdMaxSegments && plan.avg_len <= kTileBwdMaxLen)) &&
         tile_layer_bwd_supported(gather_stride(ctx->dims[layer - 1], ctx->dims[layer]), ctx->dims[layer - 1], ctx->layer_kind == 1);
}

// The backward pass of a mean-aggregator layer that shrinks: the transposed aggregate at the output width, then
// [mean^T dZ | dZ] [W_n ; W_s]^T?  (Else the products first, at twice the input width.)  Steps, us, products first / this: last layers 128 -> 47 on 306250 rows
// of 45 entries 4512 / 4172, 512 -> 100 on 89625 of 21 7426 / 7133; hidden layers of equal widths besides: 128 on 306250 rows the same, 512 on 89625 1.5 %
// and 128 on 578125 beside 308000 kept boundary rows 1 % slower (the boundary rows' product), hence an eighth narrower.  Not in layer 1, which has
// no input gradient in a step (its boundary rows need no workspace then), nor on partitions that may take the one-launch form, whose weights are
// packed as one matrix.
bool sage_gathers_first(int layer_kind, int32_t n_in, int layer, int d_in, int d_out) {
  return layer_kind == 1 && layer > 1 && d_out * 8 <= d_in * 7 && n_in > kTileBwdMaxRows;
}
bool sage_gathers_first(const bns_ctx *ctx, int layer) {
  return sage_gathers_first(ctx->layer_kind, ctx->part.n_in, layer, ctx->dims[layer - 1], ctx->dims[layer]);
}

// The forward product of `layer` by splits (gemm.hip) instead of the fp32 chain?  It is faster and closer to the exact sums (2-norm of
// the error, normal operands, beside the chain: depth 128 0.6e-7 and 2.0e-7, 256 0.7 and 2.9, 512 0.9 and 4.1, 602 1.0 and 4.4).
// Only the last layer's: sums in another order switch hidden units within rounding of zero, and one such unit of a node
// with few neighbours is a visible part of the gradient of the boundary nodes next to it.  Within a step no unit hangs on the logits; their last
// bits reach the weights through the gradients, and there they do what those of the weight gradients' sums do: a unit of a later epoch may
// switch (ten epochs from the same start, by splits and by the chain, largest difference of a gradient over its rms: 306250 rows
// 3e-6, 89625 rows with 512 hidden units 5e-6 up to the second epoch, 0.03 in the fourth).  A layer that may run as one launch has the
// bits of the chain there.  Up to a depth (d_in, also where the mean aggregator's product is twice as deep) of 64 the stores bound either.
// Products in a step, chain and splits, us: 578125 rows, 256 -> 172 542 and 338,
// 89625 rows, 1024 -> 100 218 and 117, 110645 of 512 -> 100 151 and 87, 226887 of 256 -> 41 78 and 62.
bool fwd_by_splits(const bns_ctx *ctx, int layer) {
  return layer + 1 == (int)ctx->dims.size() && ctx->dims[layer - 1] > 64 && !tile_layer(ctx, layer);
}
hipError_t fwd_product(const bns_ctx *ctx, int layer, const RowsF32 &g, const float *W, hipStream_t s) {
  return fwd_by_splits(ctx, layer) ? gemm_fwd_split(g, W, s) : gemm_rows_f32(g, s);
}
// Bytes of the first of the two matrices of a layer whose halves are packed apart.
size_t packed_fwd_half(const bns_ctx *ctx, int layer) {
  const int d_in = ctx->dims[layer - 1], d_out = ctx->dims[layer];
  return fwd_by_splits(ctx, layer) ? packed_bytes(d_in, d_out) : packed_bytes_f32(d_in, d_out);
}

bool valid_desc(const bns_partition_desc *p, const bns_model_desc *m) {
  if (!p || !m || !m->dims) return false;
  if (p->n_in < 1 || p->n_halo < 0 || p->nnz0 < p->n_in || p->e_in < p->n_in || p->e_bd < 0) return false;
  if (p->e_in + p->e_bd != p->nnz0) return false;
  if (m->n_layers < 1 || (m->loss_kind != 0 && m->loss_kind != 1)) return false;
  if (m->layer_kind != 0 && m->layer_kind != 1) return false;
  for (int l = 0; l <= m->n_layers; ++l) {
    // The aggregate holds a row in at most 8 pieces of 64 lanes x 4 floats.  The lower limits of the other widths are from when their
    // lanes took 2 floats or 1; no wider row of theirs has been tested.
    const int d = m->dims[l], cap = d % 4 == 0 ? 2048 : d % 2 == 0 ? 1024 : 512;
    if (d < 1 || d > cap) return false;
  }
  return true;
}

bool fits_int32(const bns_partition_desc *p, const bns_model_desc *m) {
  const int64_t lim = INT32_MAX;
  if (p->nnz0 >= lim || (int64_t)p->n_in + p->n_halo + 1 >= lim) return false;
  int64_t dmax = 0;
  for (int l = 0; l <= m->n_layers; ++l) dmax = std::max<int64_t>(dmax, m->dims[l]);
  return ((int64_t)p->n_in + p->n_halo) * dmax < (int64_t)1 << 40;  // byte offsets are 64-bit
}

size_t carve(Carver &c, const bns_partition_desc *p, const bns_model_desc *m, Layout *out) {
  const size_t n_in = p->n_in, B = p->n_halo, L = m->n_layers;
  size_t d_max = 0, d_out_max = 0, d_first_max = 0;  // d_out_max: of the layers whose boundary rows have a gradient of that width
  for (size_t l = 0; l <= L; ++l) d_max = std::max<size_t>(d_max, m->dims[l]);
  for (size_t l = 0; l < L; ++l) {
    if (m->layer_kind == 0 ? m->dims[l + 1] < m->dims[l] : sage_gathers_first(m->layer_kind, p->n_in, (int)l + 1, m->dims[l], m->dims[l + 1])) d_out_max = std::max<size_t>(d_out_max, m->dims[l + 1]);
    if (update_first_shape(m->layer_kind, m->dims[l], m->dims[l + 1]))
      d_first_max = std::max<size_t>(d_first_max, gather_stride(m->dims[l], m->dims[l + 1]));
  }
  Layout w;
  w.dis_in = c.take<float>(n_in);
  w.dis_halo = c.take<float>(B);
  w.split.n_inner = c.take<int32_t>(n_in);
  w.split.inner_ptr = c.take<int32_t>(n_in + 1);
  w.split.bd_ptr = c.take<int32_t>(n_in + 1);
  w.split.in_col = c.take<int32_t>(p->e_in);
  w.split.in_bdp = c.take<int32_t>(p->e_in);
  w.split.bd_b = c.take<int32_t>(p->e_bd);
  w.split.bd_row = c.take<int32_t>(p->e_bd);
  w.tile_sums = c.take<int32_t>(scan_tiles(p->nnz0 + n_in + B) + 4);
  w.kept_start = c.take<int32_t>((int64_t)B + 1);
  w.ballots = c.take<uint64_t>((B + 63) / 64 + 1);
  w.bd_mask = c.take<uint64_t>((p->e_bd + 63) / 64);
  w.bd_sums = c.take<int32_t>(scan_tiles(p->e_bd));
  w.bd_before = c.take<int32_t>((p->e_bd + 63) / 64);
  w.Hu = c.take<float>(B * d_out_max);
  w.Hu2 = c.take<float>(B * d_first_max);
  w.halo_rec = c.take<int2>(B + 1);
  w.G0 = c.take<float>(n_in * d_max);
  w.G1 = c.take<float>(n_in * d_max);
  w.G2 = c.take<float>(n_in * d_max);
  w.inv_deg = c.take<float>(n_in);
  w.w_fwd = m->layer_kind == 0 ? c.take<float>(p->e_in) : nullptr;
  w.w_bwd = c.take<float>(p->e_in);
  w.w_halo = c.take<float>(p->e_bd);
  w.loss_partials = c.take<float>(kLossBlocks);
  for (int k = 0; k < 2; ++k) {
    SegPlan &pl = k == 0 ? w.plan_f : w.plan_b;
    const int64_t nnz = k == 0 ? p->nnz0 : p->e_in;
    pl.seg_ptr = c.take<int32_t>(n_in + 1);
    pl.seg_unit = c.take<int2>(seg_max_segments(n_in, nnz));
    pl.part_ptr = c.take<int32_t>(n_in + 1);
    pl.mrow = c.take<int32_t>(seg_max_multi(nnz));
    pl.part_unit = c.take<int2>(seg_max_parts(nnz));
    pl.order = c.take<int2>(seg_max_segments(n_in, nnz));
    pl.arrived = c.take<int32_t>(4 * seg_max_parts(nnz));
    pl.n_seg = pl.n_part = pl.n_multi = 0;
  }
  w.seg_tmp_a = c.take<int32_t>(n_in + 1);
  w.seg_tmp_b = c.take<int32_t>(n_in + 2);
  w.spmm_partials = c.take<float>((size_t)seg_max_parts(p->nnz0) * d_max);
  w.C0 = c.take<float>(n_in * (size_t)m->dims[0]);
  w.kept_ids = c.take<int32_t>(B + 1);
  w.remap = c.take<int32_t>(B + 1);
  w.counters = c.take<int32_t>(64);
  w.row_ptr = c.take<int32_t>(n_in + 1);
  w.col_idx = c.take<int32_t>(p->nnz0);
  w.t_row_ptr = c.take<int32_t>(n_in + B + 1);
  w.t_col_idx = c.take<int32_t>(p->nnz0);
  w.A.assign(L + 1, nullptr);
  w.H.assign(L + 1, nullptr);
  w.dZ.assign(L + 1, nullptr);
  w.Wf.assign(L + 1, nullptr);
  w.Wb.assign(L + 1, nullptr);
  w.tn.assign(L + 1, nullptr);
  w.tn2.assign(L + 1, nullptr);
  w.G_in.assign(L + 1, nullptr);
  w.G_halo.assign(L + 1, nullptr);
  std::vector<size_t> behind(L + 1, 0);
  bool hu2_taken = false;
  for (size_t l = 1; l <= L; ++l) {
    const int32_t kw = m->layer_kind == 1 ? 2 : 1;
    size_t wf_bytes = 0;
    const bool first = update_first_shape(m->layer_kind, m->dims[l - 1], m->dims[l]);
    w.tn[l] = c.take<float>(std::max(gemm_tn_partials(kw * m->dims[l - 1], m->dims[l], p->n_in, 0),
                                     first ? gemm_tn_partials(m->dims[l - 1], m->dims[l], p->n_in, p->n_halo) : 0));
    if (first) {
      w.tn2[l] = c.take<float>(gemm_tn_partials(m->dims[l - 1], m->dims[l], p->n_halo, p->n_in));
      // what the forward pass leaves free, where it is enough: the rest of A[l] behind H W, and the boundary rows H_U W
      // (one buffer for all layers: for the first such layer)
      behind[l] = align_up(n_in * gather_stride(m->dims[l - 1], m->dims[l]) * sizeof(float)) / sizeof(float);
      if (behind[l] + n_in * m->dims[l] > n_in * (size_t)m->dims[l - 1]) behind[l] = 0;
      if (!behind[l]) w.G_in[l] = c.take<float>(n_in * m->dims[l]);
      if (hu2_taken) w.G_halo[l] = c.take<float>(B * m->dims[l]);
      else w.G_halo[l] = w.Hu2;
      hu2_taken = true;
    }
    for (const int32_t k : {kw * m->dims[l - 1], m->dims[l - 1]}) {  // one product or two, by either instruction
      const int32_t n = kw * m->dims[l - 1] / k;
      wf_bytes = std::max({wf_bytes, n * packed_bytes_f32(k, m->dims[l]), n * packed_bytes(k, m->dims[l])});
    }
    w.Wf[l] = c.take<char>(wf_bytes);
    w.Wb[l] = c.take<char>(kw * packed_bytes(m->dims[l], m->dims[l - 1]));
    w.A[l] = c.take<float>(n_in * (size_t)m->dims[l - 1]);
    if (behind[l] && w.A[l]) w.G_in[l] = w.A[l] + behind[l];
    w.H[l] = c.take<float>(n_in * (size_t)m->dims[l]);
    w.dZ[l] = c.take<float>(n_in * (size_t)m->dims[l]);
  }
  if (out) *out = w;
  return c.off;
}

bns_status fail(bns_ctx *ctx, bns_status st, const std::string &msg) {
  if (ctx) ctx->err = msg;
  return st;
}

bns_status hip_fail(bns_ctx *ctx, const char *what, hipError_t e) {
  // the runtime also keeps a failed call's code as its "last error": take it away, or the next
  // launcher's hipGetLastError() would report this failure once more as its own
  (void)hipGetLastError();
  return fail(ctx, BNS_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define BNS_TRY(what, expr)                                   \
  do {                                                        \
    hipError_t _e = (expr);                                   \
    if (_e != hipSuccess) return hip_fail(ctx, what, _e);     \
  } while (0)

// A launch that carries work of two kinds is taken apart while the phase that it would be counted for is timed.
bool timed(const bns_ctx *ctx, int phase) { return ((ctx->prof.mask >> phase) & 1u) && ctx->prof.used < ctx->prof.start.size(); }

// Brackets the kernels enqueued during its lifetime with two events (only if the phase is enabled).
struct PhaseTimer {
  Profiler *p = nullptr;
  hipStream_t s;
  size_t slot = 0;
  PhaseTimer(bns_ctx *ctx, int phase, hipStream_t stream) : s(stream) {
    Profiler &pr = ctx->prof;
    if (!((pr.mask >> phase) & 1u) || pr.used >= pr.start.size()) return;
    p = &pr;
    slot = pr.used++;
    pr.phase[slot] = phase;
    (void)hipEventRecord(pr.start[slot], s);
  }
  ~PhaseTimer() {
    if (p) (void)hipEventRecord(p->stop[slot], s);
  }
};

bool bad_p(double p) { return !(p >= 0.0 && p <= 1.0); }
// Kept boundary nodes to be expected: launches are shaped for it, buffers for all of them.
int32_t expected_kept(const bns_ctx *ctx, double p) { return (int32_t)std::ceil(p * ctx->part.n_halo); }
// Entries per row of a transposed aggregate, to be expected.
int32_t transposed_len(const bns_ctx *ctx, double p, bool halo_rows) {
  const bns_partition_desc &P = ctx->part;
  const double q = halo_rows ? p : 0.0;
  return (int32_t)(((double)P.e_in + q * (double)P.e_bd) / ((double)P.n_in + q * P.n_halo));
}
float halo_scale(double p) { return p > 0.0 ? (float)(1.0 / p) : 0.f; }  // 1/p is never formed at p = 0

// Dropout of hidden layer `layer` in an epoch (off when the rate is 0 or the layer has no ReLU).
Dropout dropout_of(const bns_ctx *ctx, int layer, bool relu, uint64_t seed, uint32_t epoch, const uint32_t *epoch_dev) {
  Dropout d;
  if (!relu || ctx->drop_q <= 0.0) return d;
  d.threshold = (uint64_t)std::floor((1.0 - ctx->drop_q) * 4294967296.0);
  d.scale = (float)(1.0 / (1.0 - ctx->drop_q));
  d.k0 = (uint32_t)seed;
  d.k1 = (uint32_t)(seed >> 32) ^ 0x64726F70u;
  d.c2 = ((uint32_t)ctx->part.part_id << 8) | (uint32_t)layer;
  d.epoch = epoch;
  d.epoch_dev = epoch_dev;
  return d;
}
// In that of the latest sample.
Dropout dropout_of(const bns_ctx *ctx, int layer, bool relu) {
  return dropout_of(ctx, layer, relu, ctx->cur_seed, ctx->cur_epoch, ctx->cur_epoch_dev);
}
// Slope of a surviving hidden unit: 1/(1-q) under dropout, else 1.
float mask_scale_of(const bns_ctx *ctx) {
  return ctx->drop_q > 0.0 ? (float)(1.0 / (1.0 - ctx->drop_q)) : 1.f;
}

// How bns_train_step runs the forward pass of `layer` when its first-layer input is X.
int layer_plan(const bns_ctx *ctx, int layer, const float *X) {
  const int d_in = ctx->dims[layer - 1], d_out = ctx->dims[layer];
  const bool cached = layer == 1 && ctx->cache_X != nullptr && ctx->cache_X == X;
  // worth its extra launches only when the aggregate is big: at least 2^24 fewer floats gathered
  const bool big = (int64_t)ctx->part.nnz0 * (d_in - d_out) >= ((int64_t)1 << 24);
  if (!cached && big && update_first_shape(ctx->layer_kind, d_in, d_out)) return BNS_LAYER_UPDATE_FIRST;
  if (one_kernel_layer(ctx, d_in, d_out)) return BNS_LAYER_ONE_KERNEL;
  return BNS_LAYER_TWO_KERNELS;
}

// update_first: H_out = act(P [H_in W ; Hu W]) instead of act((P [H_in ; Hu]) W); A_saved then
// receives H_in W (the aggregate of the inputs is never formed).  prepare (nullable): the weights to pack, when
// neither they nor the boundary records are ready.  loss (nullable): of the last layer's output; where it is formed on the way,
// its n_partials is set.
bns_status layer_fwd_impl(bns_ctx *ctx, int layer, double p, const float *H_in, const float *halo_h,
                          const float *W, float *A_saved, float *H_out, bool relu, bool update_first,
                          const PackJobs *prepare, TileLoss *loss, hipStream_t s) {
  const int n_in = ctx->part.n_in, B = ctx->part.n_halo;
  const int d_in = ctx->dims[layer - 1], d_out = ctx->dims[layer];
  const bool sage = ctx->layer_kind == 1;
  if (update_first) {
    const int ld = gather_stride(d_in, d_out);  // row stride of H W and H_U W
    {
      PhaseTimer t(ctx, BNS_PHASE_GEMM_FWD, s);
      RowsF32 g{};
      g.M = n_in;
      g.N = d_out;
      g.K = g.lda = d_in;
      g.A = H_in;
      g.Bp = ctx->ws.Wf[layer];
      g.C = A_saved;
      g.ldc = ld;
      g.pad = ld != d_out;
      if (B > 0) {  // the kept boundary rows where the caller holds them, scaled on their way in
        g.rec = ctx->ws.halo_rec;
        g.A_rec = halo_h;
        g.C_rec = ctx->ws.Hu2;
        g.M2 = B;
        g.m2_expected = expected_kept(ctx, p);
        g.m2_dev = ctx->cur_n_kept;
      }
      BNS_TRY("fwd_product", fwd_product(ctx, layer, g, W, s));
    }
    PhaseTimer t(ctx, BNS_PHASE_SPMM_FWD, s);
    BNS_TRY("spmm_fwd", spmm_fwd(ctx->ws.plan_f, n_in, ld, ctx->cur_row_ptr, ctx->cur_col_idx, ctx->ws.w_fwd,
                                 ctx->ws.split.inner_ptr, ctx->ws.dis_in, A_saved, ctx->ws.Hu2, ctx->ws.spmm_partials, H_out, SpmmRowPart{},
                                 false, relu, s, d_out));
    BNS_TRY("dropout_inplace", dropout_inplace(n_in, d_out, H_out, dropout_of(ctx, layer, relu), s));
    return BNS_OK;
  }
  // The aggregate reads the kept boundary rows where the caller holds them; it only needs, per
  // kept node, the row index and the weight S_uu = 1/p (GCN: times d~^-1/2).  A gathered, scaled
  // copy of the rows would cost a read and a write of every kept row on top of the same reads.
  // In a training step the sampler has written these records and the weights are packed.
  if (prepare) {
    const bool apart = timed(ctx, BNS_PHASE_GATHER);
    if (apart) BNS_TRY("pack_weights", pack_weights(*prepare, s));
    PhaseTimer t(ctx, BNS_PHASE_GATHER, s);
    BNS_TRY("halo_records", halo_records(ctx->cur_kept, ctx->cur_n_kept, B, sage ? nullptr : ctx->ws.dis_halo,
                                         halo_scale(p), ctx->ws.halo_rec, apart ? PackJobs{} : *prepare, s));
  }
  SpmmRowPart part;
  part.halo_rec = B > 0 ? ctx->ws.halo_rec : nullptr;
  part.skip_self = sage;
  if (layer == 1 && ctx->cache_X != nullptr && ctx->cache_X == H_in) {
    // inner neighbours are the same every epoch: their sum is cached, only the kept boundary
    // tail of each row is aggregated now
    part.row_skip = ctx->ws.split.n_inner;
    part.init = ctx->ws.C0;
  }
  const float *w_in = ctx->ws.w_fwd;
  const int32_t *w_ptr = ctx->ws.split.inner_ptr;
  const float *row_scale = sage ? ctx->ws.inv_deg : ctx->ws.dis_in;
  if (one_kernel_layer(ctx, d_in, d_out)) {
    // aggregate and update in one kernel; the partial sums of the rows cut into several segments come first
    {
      PhaseTimer t(ctx, BNS_PHASE_SPMM_LONG, s);
      BNS_TRY("spmm_fwd(long rows)", spmm_fwd(ctx->ws.plan_f, n_in, d_in, ctx->cur_row_ptr, ctx->cur_col_idx, w_in, w_ptr,
                                              row_scale, H_in, halo_h, ctx->ws.spmm_partials, A_saved, part,
                                              true, false, s));
    }
    PhaseTimer t(ctx, BNS_PHASE_SPMM_FWD, s);
    BNS_TRY("spmm_gemm_fwd", spmm_gemm_fwd(ctx->ws.plan_f, n_in, d_in, d_out, ctx->cur_row_ptr, ctx->cur_col_idx,
                                           w_in, w_ptr, row_scale, H_in, halo_h, ctx->ws.spmm_partials, A_saved,
                                           part, W, H_out, relu, dropout_of(ctx, layer, relu), s, sage));
    return BNS_OK;
  }
  if (tile_layer(ctx, layer) && !timed(ctx, BNS_PHASE_SPMM_FWD) && !timed(ctx, BNS_PHASE_GEMM_FWD)) {
    const size_t n_w = (size_t)(sage ? 2 : 1) * d_in * d_out, n_a = (size_t)n_in * d_in, n_h = (size_t)n_in * d_out;
    const auto meets = [&](const float *out, size_t n) {  // (one kernel reads what two have read before the second writes)
      return overlap(out, n, H_in, n_a) || overlap(out, n, halo_h, (size_t)B * d_in) || overlap(out, n, W, n_w);
    };
    if (!meets(A_saved, n_a) && !meets(H_out, n_h)) {
      BNS_TRY("tile_layer_fwd", tile_layer_fwd(ctx->ws.plan_f, n_in, d_in, d_out, ctx->cur_row_ptr, ctx->cur_col_idx, w_in, w_ptr,
                                               row_scale, H_in, halo_h, ctx->ws.spmm_partials, A_saved, part, W, H_out, relu,
                                               dropout_of(ctx, layer, relu), sage, concat_in_one(d_in),
                                               loss && d_out <= kTileLossWidth && !timed(ctx, BNS_PHASE_LOSS) ? loss : nullptr, s));
      return BNS_OK;
    }
  }
  {
    PhaseTimer t(ctx, BNS_PHASE_SPMM_FWD, s);
    BNS_TRY("spmm_fwd", spmm_fwd(ctx->ws.plan_f, n_in, d_in, ctx->cur_row_ptr, ctx->cur_col_idx, w_in, w_ptr, row_scale,
                                 H_in, halo_h, ctx->ws.spmm_partials, A_saved, part, false, false, s));
  }
  {
    PhaseTimer t(ctx, BNS_PHASE_GEMM_FWD, s);
    RowsF32 g{};
    g.M = n_in;
    g.N = g.ldc = d_out;
    g.K = g.lda = d_in;
    g.A = A_saved;
    g.Bp = ctx->ws.Wf[layer];
    g.C = H_out;
    if (sage && concat_in_one(d_in)) {  // [z | h] [W_n ; W_s] in one product
      g.A2 = H_in;
      g.a_split = d_in;
      g.K = 2 * d_in;
    } else if (sage) {  // z W_n + h W_s
      BNS_TRY("fwd_product(nbr)", fwd_product(ctx, layer, g, W, s));
      W += (size_t)d_in * d_out;
      g.A = H_in;
      g.Bp = ctx->ws.Wf[layer] + packed_fwd_half(ctx, layer);
      g.accumulate = true;
    }
    g.relu = relu;
    g.drop = dropout_of(ctx, layer, relu);
    BNS_TRY("fwd_product(update)", fwd_product(ctx, layer, g, W, s));
  }
  return BNS_OK;
}

// Does the backward pass of `layer` gather its dZ at the output width, in padded rows?
bool pads_gradient(const bns_ctx *ctx, int layer, double p, bool update_first, bool input_gradient) {
  const int d_in = ctx->dims[layer - 1], d_out = ctx->dims[layer];
  if (gather_stride(d_in, d_out) == d_out) return false;
  return update_first || ((ctx->layer_kind == 0 || sage_gathers_first(ctx, layer) || tile_layer_bwd(ctx, layer, ctx->part.n_in + (int64_t)expected_kept(ctx, p))) && input_gradient && d_out < d_in);
}

// The weight gradients of several layers, to be run together.
struct TnBatch {
  TnGemm g[kMaxTnJobs];
  int n = 0;
  bool full() const { return n + 2 > kMaxTnJobs; }
};
bns_status run_batch(bns_ctx *ctx, TnBatch *batch, const TnLoss &loss, hipStream_t s) {
  PhaseTimer t(ctx, BNS_PHASE_GEMM_DW, s);
  BNS_TRY("gemm_tn", gemm_tn(batch->g, batch->n, loss, s));
  batch->n = 0;
  return BNS_OK;
}

// dZ is the gradient of the layer's pre-activation.  mask_src (nullable): activations of the
// layer below; when given, dH_in receives the masked gradient (= dZ of the layer below).
// H_in is needed by the mean-aggregator layer only (its self half of the weight gradient).
// halo_first (nullable): the boundary features of an update-first layer (A_saved does not hold
// the aggregate then); the weight gradient is [H_in ; Hu]^T (P^T dZ) instead of A^T dZ.
// dz_padded: G2 holds dZ with padded rows already (pads_gradient).
// sage_first: the weights are packed for sage_gathers_first, and neither dH_in nor dhalo shares memory with dZ or W.
// batch (nullable): collects the weight gradient, to be run when the chain of the layers is through; without one it is
// run before dH_in and dhalo are written, which may then share memory with dZ, A_saved or H_in.
bns_status layer_bwd_impl(bns_ctx *ctx, int layer, double p, const float *dZ, const float *A_saved,
                          const float *H_in, const float *W, float *dW, float *dH_in, float *dhalo, const float *mask_src,
                          bool update_first, const float *halo_first, float *W_step, float lr, bool dz_padded,
                          bool sage_first, TnBatch *batch, hipStream_t s) {
  const int n_in = ctx->part.n_in, B = ctx->part.n_halo;
  const int d_in = ctx->dims[layer - 1], d_out = ctx->dims[layer];
  const char *Wb = ctx->ws.Wb[layer];
  // C = alpha * G W^T for the inner rows of G at the output width; C2: the mean aggregator's second half; G_more: the
  // rows of the kept boundary nodes; G2: times the second half of W, added to C
  auto gemm_wt = [&](const float *G, float *C, float *C2, const float *mask, float alpha, const float *G_more, float *C_more, const float *G2 = nullptr) {
    RowsGemm g{};
    g.M = n_in;
    g.N = C2 ? 2 * d_in : d_in;
    g.K = g.lda = d_out;
    g.A = G;
    g.A2 = G2;
    g.W = W;
    g.Bp = Wb;
    g.C = C;
    g.alpha = alpha;
    if (C2 && d_in % 4 != 0) {  // no 16-byte store may straddle the two results: one product each
      g.N = g.ldc = d_in;
      const hipError_t e = gemm_rows(g, s);
      if (e != hipSuccess) return e;
      g.W = W + (size_t)d_in * d_out;
      g.Bp = Wb + packed_bytes(d_out, d_in);
      g.C = C2;
      return gemm_rows(g, s);
    }
    g.C2 = C2;
    g.ldc = g.c_split = d_in;
    g.mask = mask;
    g.A_more = G_more;
    g.C_more = C_more;
    g.M2 = B;
    g.m2_expected = expected_kept(ctx, p);
    g.m2_dev = ctx->cur_n_kept;
    return gemm_rows(g, s);
  };
  TnBatch own;
  TnBatch *const jobs = batch ? batch : &own;
  auto add_dw = [&](int32_t K, const float *A, const float *A2, const float *G, float *partials) {  // dW = [A | A2]^T G
    TnGemm &g = jobs->g[jobs->n++];
    g = TnGemm{};
    g.M = A2 ? 2 * d_in : d_in;
    g.N = d_out;
    g.K = K;
    g.A = A;
    g.A2 = A2;
    g.B = G;
    g.a_split = d_in;
    g.C = dW;
    g.partials = partials;
    g.W = W_step;
    g.lr = lr;
    return &g;
  };
  if (update_first) {
    float *G_in = ctx->ws.G_in[layer], *G_halo = B > 0 ? ctx->ws.G_halo[layer] : nullptr;
    {  // G = P^T dZ at the output width, inner rows and kept boundary rows
      PhaseTimer t(ctx, BNS_PHASE_SPMM_BWD, s);
      const int ld = gather_stride(d_in, d_out);
      const float *dZ_g = dZ;
      if (ld != d_out) {  // the gathered operand with padded rows
        if (!dz_padded) BNS_TRY("pad_rows", pad_rows(n_in, d_out, ld, dZ, ctx->ws.G2, s));
        dZ_g = ctx->ws.G2;
      }
      BNS_TRY("spmm_bwd", spmm_bwd(ctx->ws.plan_b, n_in, B, ld, ctx->cur_t_row_ptr, ctx->cur_t_col_idx,
                                   ctx->cur_kept, ctx->cur_n_kept, ctx->ws.w_bwd, ctx->ws.w_halo, ctx->part.halo_ptr, ctx->ws.dis_in,
                                   ctx->ws.dis_halo,
                                   halo_scale(p), dZ_g, nullptr, nullptr, false, transposed_len(ctx, p, G_halo), ctx->ws.spmm_partials, G_in, G_halo,
                                   expected_kept(ctx, p), s, d_out));
    }
    add_dw(n_in, H_in, nullptr, G_in, ctx->ws.tn[layer]);
    if (B > 0) {  // the kept boundary features where the caller holds them: G_halo carries the 1/p and degree factors
      TnGemm *g = add_dw(B, halo_first, nullptr, G_halo, ctx->ws.tn2[layer]);
      g->rows = ctx->cur_kept;
      g->k_dev = ctx->cur_n_kept;
      g->k_expected = expected_kept(ctx, p);
      g->accumulate = true;
    }
    if (dH_in) {
      PhaseTimer t(ctx, BNS_PHASE_GEMM_DA, s);
      const float ms1 = mask_src ? mask_scale_of(ctx) : 1.f;
      BNS_TRY("gemm_rows(dH)", gemm_wt(G_in, dH_in, nullptr, mask_src, ms1, dhalo ? G_halo : nullptr, dhalo));
    }
    return BNS_OK;
  }
  // slope of the surviving hidden units of the layer below (dropout); it multiplies the masked
  // gradient only.  Where the transposed aggregate applies the mask, the factor rides on its
  // input (the product with W^T) and is divided out of the boundary rows, which are not masked.
  const float ms = mask_src ? mask_scale_of(ctx) : 1.f;
  // mean aggregator: [A | H]^T dZ in one product, dZ is read once
  add_dw(n_in, A_saved, ctx->layer_kind == 1 ? H_in : nullptr, dZ, ctx->ws.tn[layer]);
  if (!batch) {
    const bns_status st = run_batch(ctx, &own, TnLoss{}, s);
    if (st != BNS_OK) return st;
  }
  const int ld_g = gather_stride(d_in, d_out);
  if (dH_in && tile_layer_bwd(ctx, layer, n_in + (dhalo ? (int64_t)expected_kept(ctx, p) : 0)) && !timed(ctx, BNS_PHASE_SPMM_BWD) && !timed(ctx, BNS_PHASE_GEMM_DA) &&
      (ld_g == d_out || dz_padded || ctx->layer_kind == 0)) {
    const size_t n_w = (size_t)(ctx->layer_kind == 1 ? 2 : 1) * d_in * d_out, n_h = (size_t)n_in * d_in;
    const auto meets = [&](const float *out, size_t n) {
      return overlap(out, n, dZ, (size_t)n_in * d_out) || overlap(out, n, W, n_w) || (mask_src && overlap(out, n, mask_src, n_h));
    };
    if (!meets(dH_in, n_h) && !(dhalo && meets(dhalo, (size_t)B * d_in))) {
      if (ld_g != d_out && !dz_padded) BNS_TRY("pad_rows", pad_rows(n_in, d_out, ld_g, dZ, ctx->ws.G2, s));
      const bool gcn = ctx->layer_kind == 0;
      BNS_TRY("tile_layer_bwd", tile_layer_bwd(ctx->ws.plan_b, n_in, B, ld_g, d_in, d_out, ctx->cur_t_row_ptr, ctx->cur_t_col_idx,
                                               ctx->cur_kept, ctx->cur_n_kept, ctx->ws.w_bwd, ctx->ws.w_halo, ctx->part.halo_ptr,
                                               gcn ? ctx->ws.dis_in : nullptr, gcn ? ctx->ws.dis_halo : nullptr, halo_scale(p),
                                               ld_g != d_out ? ctx->ws.G2 : dZ, W, Wb, mask_src, ms, !gcn, ctx->ws.spmm_partials,
                                               dH_in, dhalo, expected_kept(ctx, p), s));
      return BNS_OK;
    }
  }
  if (ctx->layer_kind == 1 && !sage_first) {
    if (dH_in) {
      {
        PhaseTimer t(ctx, BNS_PHASE_GEMM_DA, s);  // dZ [W_n ; W_s]^T in one product, split into the two halves
        BNS_TRY("gemm_rows(dA pair)", gemm_wt(dZ, ctx->ws.G1, ctx->ws.G2, nullptr, ms, nullptr, nullptr));
      }
      // dH_in = (gradient through the node's own feature) + mean^T (gradient of the neighbour mean)
      PhaseTimer t(ctx, BNS_PHASE_SPMM_BWD, s);
      BNS_TRY("spmm_bwd", spmm_bwd(ctx->ws.plan_b, n_in, B, d_in, ctx->cur_t_row_ptr, ctx->cur_t_col_idx,
                                   ctx->cur_kept, ctx->cur_n_kept, ctx->ws.w_bwd, ctx->ws.w_halo, ctx->part.halo_ptr, nullptr, nullptr,
                                   halo_scale(p) / ms, ctx->ws.G1, mask_src, ctx->ws.G2, true,
                                   transposed_len(ctx, p, dhalo), ctx->ws.spmm_partials, dH_in, dhalo, expected_kept(ctx, p), s));
    }
    return BNS_OK;
  }
  if (dH_in && d_out < d_in) {
    // (P^T dZ) W^T instead of P^T (dZ W^T): the transposed aggregate runs at the narrower width (mean aggregator: and half as much is
    // written and read between the launches)
    const bool sage = ctx->layer_kind == 1;
    float *G_in = ctx->ws.G1, *G_halo = dhalo && B > 0 ? ctx->ws.Hu : nullptr;
    {
      PhaseTimer t(ctx, BNS_PHASE_SPMM_BWD, s);
      const int ld = gather_stride(d_in, d_out);
      const float *dZ_g = dZ;
      if (ld != d_out) {  // the gathered operand with padded rows
        if (!dz_padded) BNS_TRY("pad_rows", pad_rows(n_in, d_out, ld, dZ, ctx->ws.G2, s));
        dZ_g = ctx->ws.G2;
      }
      BNS_TRY("spmm_bwd", spmm_bwd(ctx->ws.plan_b, n_in, B, ld, ctx->cur_t_row_ptr, ctx->cur_t_col_idx,
                                   ctx->cur_kept, ctx->cur_n_kept, ctx->ws.w_bwd, ctx->ws.w_halo, ctx->part.halo_ptr, sage ? nullptr : ctx->ws.dis_in,
                                   sage ? nullptr : ctx->ws.dis_halo, halo_scale(p), dZ_g, nullptr, nullptr, sage,
                                   transposed_len(ctx, p, G_halo), ctx->ws.spmm_partials, G_in, G_halo, expected_kept(ctx, p), s, d_out));
    }
    PhaseTimer t(ctx, BNS_PHASE_GEMM_DA, s);
    BNS_TRY("gemm_rows(dH)", gemm_wt(G_in, dH_in, nullptr, mask_src, ms, G_halo, dhalo, sage ? dZ : nullptr));
  } else if (dH_in) {
    {
      PhaseTimer t(ctx, BNS_PHASE_GEMM_DA, s);
      BNS_TRY("gemm_rows(dA)", gemm_wt(dZ, ctx->ws.G1, nullptr, nullptr, ms, nullptr, nullptr));
    }
    PhaseTimer t(ctx, BNS_PHASE_SPMM_BWD, s);
    BNS_TRY("spmm_bwd", spmm_bwd(ctx->ws.plan_b, n_in, B, d_in, ctx->cur_t_row_ptr, ctx->cur_t_col_idx,
                                 ctx->cur_kept, ctx->cur_n_kept, ctx->ws.w_bwd, ctx->ws.w_halo, ctx->part.halo_ptr, ctx->ws.dis_in,
                                 ctx->ws.dis_halo, halo_scale(p) / ms, ctx->ws.G1, mask_src, nullptr, false,
                                 transposed_len(ctx, p, dhalo), ctx->ws.spmm_partials, dH_in, dhalo, expected_kept(ctx, p), s));
  }
  return BNS_OK;
}

// Adds the weights of layer l to the packing jobs, for the forward product and / or for dZ W^T.
// halves: the layer's backward pass is that of sage_gathers_first.
void add_pack_jobs(const bns_ctx *ctx, int l, const float *W, bool fwd, bool bwd, bool halves, PackJobs *jobs) {
  const int32_t kw = ctx->layer_kind == 1 ? 2 : 1, d_in = ctx->dims[l - 1], d_out = ctx->dims[l];
  const size_t half = (size_t)d_in * d_out;
  auto add = [&](const float *w, char *out, int32_t K, int32_t N, bool split, bool of_fwd = false) {
    PackJob &j = jobs->j[jobs->n++];
    j = PackJob{w, out, K, N, split, of_fwd};
    jobs->units += pack_units(j);
  };
  // a layer in one kernel reads its weights as they are
  if (fwd && (!one_kernel_layer(ctx, d_in, d_out) ||
              update_first_shape(ctx->layer_kind, d_in, d_out))) {
    if (kw == 2 && !concat_in_one(d_in)) {  // the two halves apart
      add(W, ctx->ws.Wf[l], d_in, d_out, fwd_by_splits(ctx, l), true);
      add(W + half, ctx->ws.Wf[l] + packed_fwd_half(ctx, l), d_in, d_out, fwd_by_splits(ctx, l), true);
    } else {
      add(W, ctx->ws.Wf[l], kw * d_in, d_out, fwd_by_splits(ctx, l), true);
    }
  }
  if (bwd) {
    if (kw == 2 && (d_in % 4 != 0 || halves)) {  // the two halves apart (see gemm_wt)
      add(W, ctx->ws.Wb[l], d_out, d_in, true);
      add(W + half, ctx->ws.Wb[l] + packed_bytes(d_out, d_in), d_out, d_in, true);
    } else {
      add(W, ctx->ws.Wb[l], d_out, kw * d_in, true);
    }
  }
}
constexpr int kPackLayers = kMaxPackJobs / 4;  // layers whose jobs fit one launch

// Are the arrays of the workspace current and still unwritten, i.e. has a step been captured and none been run?
bool no_subgraph(const bns_ctx *ctx) { return ctx->cur_row_ptr == ctx->ws.row_ptr && !ctx->ws_built; }

BdCount bd_count(const bns_ctx *ctx) { return BdCount{ctx->part.e_bd, ctx->ws.split.bd_b, ctx->ws.bd_mask, ctx->ws.bd_sums, ctx->ws.bd_before}; }

// pack (nullable): a training step's: weights to pack beside the sampling, and the records of the kept nodes too
bns_status sample_impl(bns_ctx *ctx, uint64_t seed, uint32_t epoch, const uint32_t *epoch_dev, double p,
                       int32_t *kept_ids, int32_t *remap, int32_t *n_kept, const PackJobs *pack, hipStream_t s) {
  const uint64_t threshold = (uint64_t)std::floor(p * 4294967296.0);
  const BdCount count = bd_count(ctx);
  PhaseTimer t(ctx, BNS_PHASE_SAMPLE, s);
  BNS_TRY("sample_boundary",
          sample_boundary(ctx->part.halo_gid, ctx->part.n_halo, seed, epoch, epoch_dev, (uint32_t)ctx->part.part_id,
                          threshold, ctx->ws.ballots, ctx->ws.tile_sums, kept_ids, remap, n_kept, ctx->part.halo_ptr,
                          (int32_t)ctx->part.e_in, ctx->ws.kept_start, pack ? ctx->ws.halo_rec : nullptr,
                          ctx->layer_kind == 1 ? nullptr : ctx->ws.dis_halo, halo_scale(p), pack, &count, s));
  ctx->cur_counted = true;
  ctx->drawn = remap;
  ctx->cur_kept = kept_ids;
  ctx->cur_remap = remap;
  ctx->cur_n_kept = n_kept;
  ctx->cur_seed = seed;
  ctx->cur_epoch = epoch;
  ctx->cur_epoch_dev = epoch_dev;
  return BNS_OK;
}

bns_status build_impl(bns_ctx *ctx, int32_t *row_ptr, int32_t *col_idx, int32_t *t_row_ptr,
                      int32_t *t_col_idx, int32_t *nnz, hipStream_t s) {
  const bns_partition_desc &P = ctx->part;
  PhaseTimer t(ctx, BNS_PHASE_BUILD, s);
  SubgraphBuild g{};
  g.n_in = P.n_in; g.n_halo = P.n_halo; g.e_in = P.e_in;
  g.sp = ctx->ws.split;
  g.bd = bd_count(ctx);
  g.ballots = ctx->ws.ballots;
  g.remap = ctx->cur_remap; g.kept_ids = ctx->cur_kept; g.n_kept = ctx->cur_n_kept; g.kept_start = ctx->ws.kept_start;
  g.t_in_ptr = P.t_in_ptr; g.t_in_col = P.t_in_col; g.halo_ptr = P.halo_ptr; g.halo_col = P.halo_col;
  g.row_ptr = row_ptr; g.col_idx = col_idx; g.nnz = nnz; g.t_row_ptr = t_row_ptr; g.t_col_idx = t_col_idx;
  // the workspace arrays hold the static rows since bns_create
  g.static_rows = !(t_row_ptr == ctx->ws.t_row_ptr && t_col_idx == ctx->ws.t_col_idx);
  BNS_TRY("build_subgraph", build_subgraph(g, ctx->cur_counted, s));
  if (row_ptr == ctx->ws.row_ptr) ctx->ws_built = true;
  ctx->cur_row_ptr = row_ptr;
  ctx->cur_col_idx = col_idx;
  ctx->cur_t_row_ptr = t_row_ptr;
  ctx->cur_t_col_idx = t_col_idx;
  return BNS_OK;
}

// What the first layer of a training step reads; done: its forward pass was part of the subgraph's launch.
struct FirstLayer {
  const float *X, *halo_h, *W;
  bool done = false;
};

// The first layer's forward pass in the launch of a small partition's subgraph?  Where it would be a launch of few rows on its own (tile_layer) and has no
// rows of several segments.  Steps, two launches / one, us: 64-16-8, 400 rows 25.5 / 21.6, 64-128-47, 1000 rows of 6 entries 32.5 / 28.3,
// 100-128-128-47, 2000 of 12 64.7 / 61.9, 128-128-128-47, 3000 of 13 77.1 / 76.0, 64-256-41, 4500 of 7 75.7 / 69.6, mean aggregator 100-100-41, 2500 of 18
// 62.6 / 54.7, 128-128-41, 6000 of 5 69.9 / 70.3.  So not for rows of more than 64 floats where the tiles are of 16 rows: a compute unit holds one
// of these workgroups (85 to 101 KB of LDS), and their wavefronts have two rows each to look up and to gather.  Not while one of the phases is timed.
constexpr int kFirstWideMaxRows = 3584;  // of tile_rows
bool first_in_subgraph_launch(const bns_ctx *ctx, const FirstLayer &first) {
  if (ctx->n_layers < 2 || ctx->ws.plan_f.n_multi > 0 || layer_plan(ctx, 1, first.X) != BNS_LAYER_TWO_KERNELS || !tile_layer(ctx, 1)) return false;
  if (ctx->dims[0] > 64 && ctx->part.n_in > kFirstWideMaxRows) return false;
  for (int phase : {BNS_PHASE_SAMPLE, BNS_PHASE_BUILD, BNS_PHASE_SPMM_FWD, BNS_PHASE_GEMM_FWD})
    if (timed(ctx, phase)) return false;
  const size_t d_in = ctx->dims[0], d_out = ctx->dims[1], n_a = ctx->part.n_in * d_in, n_h = ctx->part.n_in * d_out;
  const auto meets = [&](const float *out, size_t n) {  // (as before tile_layer_fwd)
    return overlap(out, n, first.X, n_a) || overlap(out, n, first.halo_h, ctx->part.n_halo * d_in) ||
           overlap(out, n, first.W, (ctx->layer_kind == 1 ? 2 : 1) * d_in * d_out);
  };
  return !meets(ctx->ws.A[1], n_a) && !meets(ctx->ws.H[1], n_h);
}

// Selection step + subgraph step of a training step, into the workspace arrays: one launch for a
// small partition (timed as the sample phase), else the two calls above.
bns_status sample_and_build_impl(bns_ctx *ctx, uint64_t seed, uint32_t epoch, const uint32_t *epoch_dev, double p,
                                 const PackJobs &pack, FirstLayer *first, hipStream_t s) {
  Layout &w = ctx->ws;
  const bns_partition_desc &P = ctx->part;
  if (!sample_build_small_fits(P.n_in, P.n_halo, P.e_in, P.e_bd, expected_kept(ctx, p))) {
    const bns_status st = sample_impl(ctx, seed, epoch, epoch_dev, p, w.kept_ids, w.remap, w.counters, &pack, s);
    if (st != BNS_OK) return st;
    return build_impl(ctx, w.row_ptr, w.col_idx, w.t_row_ptr, w.t_col_idx, w.counters + 1, s);
  }
  const bool sage = ctx->layer_kind == 1;
  SmallArgs a;
  a.halo_gid = P.halo_gid; a.n_halo = P.n_halo;
  a.k0 = (uint32_t)seed; a.k1 = (uint32_t)(seed >> 32); a.epoch = epoch; a.epoch_dev = epoch_dev; a.part_id = (uint32_t)P.part_id;
  a.threshold = (uint64_t)std::floor(p * 4294967296.0);
  a.ballots = w.ballots; a.kept_ids = w.kept_ids; a.remap = w.remap; a.n_kept = w.counters; a.kept_start = w.kept_start;
  a.n_in = P.n_in; a.e_in = (int32_t)P.e_in; a.e_bd = (int32_t)P.e_bd;
  a.sp = w.split; a.row_ptr = w.row_ptr; a.col_idx = w.col_idx; a.nnz = w.counters + 1;
  a.halo_ptr = P.halo_ptr; a.halo_col = P.halo_col; a.t_tail_ptr = w.t_row_ptr + P.n_in; a.t_col_idx = w.t_col_idx;
  a.rec = w.halo_rec; a.dis_halo = sage ? nullptr : w.dis_halo; a.s_halo = halo_scale(p);
  first->done = first_in_subgraph_launch(ctx, *first);
  if (first->done) {
    const bool cached = ctx->cache_X != nullptr && ctx->cache_X == first->X;
    BNS_TRY("sample_build_first",
            sample_build_first(a, pack, ctx->dims[0], ctx->dims[1], w.w_fwd, sage ? w.inv_deg : w.dis_in, first->X, first->halo_h, w.A[1],
                               cached ? w.C0 : nullptr, first->W, w.H[1], true, dropout_of(ctx, 1, true, seed, epoch, epoch_dev), sage, concat_in_one(ctx->dims[0]),
                               w.plan_f, s));
  } else {
    PhaseTimer t(ctx, BNS_PHASE_SAMPLE, s);
    BNS_TRY("sample_build_small", sample_build_small(a, pack, s));
  }
  ctx->cur_counted = false;
  ctx->drawn = w.remap;
  ctx->ws_built = true;
  ctx->cur_kept = w.kept_ids;
  ctx->cur_remap = w.remap;
  ctx->cur_n_kept = w.counters;
  ctx->cur_seed = seed;
  ctx->cur_epoch = epoch;
  ctx->cur_epoch_dev = epoch_dev;
  ctx->cur_row_ptr = w.row_ptr;
  ctx->cur_col_idx = w.col_idx;
  ctx->cur_t_row_ptr = w.t_row_ptr;
  ctx->cur_t_col_idx = w.t_col_idx;
  return BNS_OK;
}

}  // namespace

extern "C" {

size_t bns_workspace_bytes(const bns_partition_desc *part, const bns_model_desc *model) {
  if (!valid_desc(part, model) || !fits_int32(part, model)) return 0;
  Carver c(nullptr);
  return carve(c, part, model, nullptr);
}

bns_status bns_create(bns_ctx **out, const bns_partition_desc *part, const bns_model_desc *model,
                      void *dev_ws, size_t ws_bytes, void *stream) {
  if (!out) return BNS_EINVAL;
  *out = nullptr;
  if (!valid_desc(part, model)) return BNS_EINVAL;
  if (!fits_int32(part, model)) return BNS_EOVERFLOW;
  if (!part->row_ptr0 || !part->col0 || !part->t_in_ptr || !part->t_in_col || !part->deg_in) return BNS_EINVAL;
  if (part->n_halo > 0 && (!part->halo_ptr || !part->halo_col || !part->halo_gid || !part->deg_halo))
    return BNS_EINVAL;
  if (!dev_ws || ((uintptr_t)dev_ws % kAlign) != 0) return BNS_EWORKSPACE;
  bns_ctx *ctx = new (std::nothrow) bns_ctx();
  if (!ctx) return BNS_EINVAL;
  ctx->part = *part;
  ctx->n_layers = model->n_layers;
  ctx->loss_kind = model->loss_kind;
  ctx->layer_kind = model->layer_kind;
  ctx->dims.assign(model->dims, model->dims + model->n_layers + 1);
  Carver c(dev_ws);
  const size_t need = carve(c, part, model, &ctx->ws);
  if (need > ws_bytes) { delete ctx; return BNS_EWORKSPACE; }
  *out = ctx;  // handed out even if set-up fails, so that the caller can read the error text
  hipStream_t s = static_cast<hipStream_t>(stream);
  BNS_TRY("degree_rsqrt(in)", degree_rsqrt(part->deg_in, part->n_in, ctx->ws.dis_in, s));
  BNS_TRY("degree_inverse", degree_inverse(part->deg_in, part->n_in, ctx->ws.inv_deg, s));
  BNS_TRY("degree_rsqrt(halo)", degree_rsqrt(part->deg_halo, part->n_halo, ctx->ws.dis_halo, s));
  BNS_TRY("build_static_split", build_static_split(part->n_in, part->row_ptr0, part->col0, ctx->ws.split,
                                                   ctx->ws.tile_sums, s));
  const float *w_col = ctx->layer_kind == 1 ? ctx->ws.inv_deg : ctx->ws.dis_in;
  if (ctx->ws.w_fwd) BNS_TRY("entry_weights(fwd)", entry_weights(part->e_in, ctx->ws.split.in_col, w_col, ctx->ws.w_fwd, s));
  BNS_TRY("entry_weights(bwd)", entry_weights(part->e_in, part->t_in_col, w_col, ctx->ws.w_bwd, s));
  BNS_TRY("entry_weights(halo)", entry_weights(part->e_bd, part->halo_col, w_col, ctx->ws.w_halo, s));
  for (const auto &[plan, nnz] : {std::pair<const SegPlan &, int64_t>(ctx->ws.plan_f, part->nnz0), std::pair<const SegPlan &, int64_t>(ctx->ws.plan_b, part->e_in)})
    BNS_TRY("clear counts", hipMemsetAsync(plan.arrived, 0, 4 * seg_max_parts(nnz) * sizeof(int32_t), s));
  int32_t *const counts = reinterpret_cast<int32_t *>(ctx->ws.spmm_partials);
  BNS_TRY("build_seg_plan(fwd)", build_seg_plan(part->n_in, part->nnz0, part->row_ptr0, part->col0, (int64_t)part->n_in + part->n_halo,
                                                 &ctx->ws.plan_f, ctx->ws.seg_tmp_a, ctx->ws.seg_tmp_b, counts, ctx->ws.tile_sums, s));
  BNS_TRY("build_seg_plan(bwd)", build_seg_plan(part->n_in, part->e_in, part->t_in_ptr, part->t_in_col, part->n_in,
                                                 &ctx->ws.plan_b, ctx->ws.seg_tmp_a, ctx->ws.seg_tmp_b, counts, ctx->ws.tile_sums, s));
  // the rows of the inner nodes in the workspace's transposed CSR are the same in every epoch
  BNS_TRY("copy_static_rows", copy_static_rows(part->n_in, part->e_in, part->t_in_ptr, part->t_in_col, ctx->ws.t_row_ptr,
                                               ctx->ws.t_col_idx, s));
  BNS_TRY("set-up sync", hipStreamSynchronize(s));
  return BNS_OK;
}

void bns_destroy(bns_ctx *ctx) {
  if (ctx && ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
  delete ctx;
}

const char *bns_last_error(const bns_ctx *ctx) {
  if (ctx) return ctx->err.c_str();
  const char *e = bns_noalloc_last_error();
  return e[0] ? e : "null context";
}

bns_status bns_sample_boundary(bns_ctx *ctx, uint64_t seed, uint32_t epoch, double p, int32_t *kept_ids,
                               int32_t *remap, int32_t *n_kept, void *stream) {
  if (!ctx) return BNS_EINVAL;
  if (bad_p(p)) return fail(ctx, BNS_EINVAL, "p must lie in [0, 1]");
  if (!n_kept || (ctx->part.n_halo > 0 && (!kept_ids || !remap)))
    return fail(ctx, BNS_EINVAL, "null output pointer");
  return sample_impl(ctx, seed, epoch, nullptr, p, kept_ids, remap, n_kept, nullptr, static_cast<hipStream_t>(stream));
}

bns_status bns_build_sampled_csr(bns_ctx *ctx, const int32_t *remap, const int32_t *kept_ids, const int32_t *n_kept,
                                 int32_t *row_ptr, int32_t *col_idx, int32_t *t_row_ptr, int32_t *t_col_idx,
                                 int32_t *nnz, void *stream) {
  if (!ctx) return BNS_EINVAL;
  if (!row_ptr || !col_idx || !t_row_ptr || !t_col_idx || !nnz)
    return fail(ctx, BNS_EINVAL, "null output pointer");
  if (!ctx->cur_n_kept) return fail(ctx, BNS_EINVAL, "bns_sample_boundary has not been called");
  // the keep bits of the latest sample sit in the workspace: the three arrays must be that sample's
  if (remap != ctx->cur_remap || kept_ids != ctx->cur_kept || n_kept != ctx->cur_n_kept)
    return fail(ctx, BNS_EINVAL, "remap / kept_ids / n_kept are not the outputs of the latest bns_sample_boundary");
  if (ctx->part.n_halo > 0 && remap != ctx->drawn)
    return fail(ctx, BNS_EINVAL, "remap / kept_ids / n_kept do not hold the latest sample: a replayed step has drawn another one since, or a captured one has not run");
  return build_impl(ctx, row_ptr, col_idx, t_row_ptr, t_col_idx, nnz, static_cast<hipStream_t>(stream));
}

bns_status bns_gcn_layer_fwd(bns_ctx *ctx, int32_t layer, double p, const float *H_in, const float *halo_h,
                             const float *W, float *A_saved, float *H_out, int32_t relu, void *stream) {
  if (!ctx) return BNS_EINVAL;
  if (layer < 1 || layer > ctx->n_layers) return fail(ctx, BNS_EINVAL, "layer out of range");
  if (bad_p(p)) return fail(ctx, BNS_EINVAL, "p must lie in [0, 1]");
  if (!H_in || !W || !A_saved || !H_out || (ctx->part.n_halo > 0 && !halo_h))
    return fail(ctx, BNS_EINVAL, "null pointer");
  if (!ctx->cur_row_ptr) return fail(ctx, BNS_EINVAL, "bns_build_sampled_csr has not been called");
  if (no_subgraph(ctx)) return fail(ctx, BNS_EINVAL, "the captured step has not run: there is no sampled subgraph yet");
  hipStream_t s = static_cast<hipStream_t>(stream);
  PackJobs jobs;
  add_pack_jobs(ctx, layer, W, true, false, false, &jobs);
  return layer_fwd_impl(ctx, layer, p, H_in, halo_h, W, A_saved, H_out, relu != 0, false, &jobs, nullptr, s);
}

bns_status bns_gcn_layer_bwd(bns_ctx *ctx, int32_t layer, double p, const float *dH_out, const float *H_out,
                             const float *A_saved, const float *H_in, const float *W, float *dW, float *dH_in,
                             float *dhalo, void *stream) {
  if (!ctx) return BNS_EINVAL;
  if (layer < 1 || layer > ctx->n_layers) return fail(ctx, BNS_EINVAL, "layer out of range");
  if (bad_p(p)) return fail(ctx, BNS_EINVAL, "p must lie in [0, 1]");
  if (!dH_out || !A_saved || !W || !dW) return fail(ctx, BNS_EINVAL, "null pointer");
  if (ctx->layer_kind == 1 && !H_in) return fail(ctx, BNS_EINVAL, "the mean-aggregator layer needs H_in");
  if (!dH_in && dhalo) return fail(ctx, BNS_EINVAL, "dhalo needs dH_in");
  if (!ctx->cur_t_row_ptr) return fail(ctx, BNS_EINVAL, "bns_build_sampled_csr has not been called");
  if (no_subgraph(ctx)) return fail(ctx, BNS_EINVAL, "the captured step has not run: there is no sampled subgraph yet");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int d_in = ctx->dims[layer - 1], d_out = ctx->dims[layer];
  const float *dZ = H_out ? ctx->ws.G0 : dH_out;
  // (the product reads dZ while it writes the two results)
  const auto meets = [&](const float *out, size_t n) { return overlap(out, n, dZ, (size_t)ctx->part.n_in * d_out) || overlap(out, n, W, (size_t)2 * d_in * d_out); };
  const bool sage_first = dH_in && sage_gathers_first(ctx, layer) && !meets(dH_in, (size_t)ctx->part.n_in * d_in) &&
                          !(dhalo && meets(dhalo, (size_t)ctx->part.n_halo * d_in));
  PackJobs jobs;
  if (dH_in) add_pack_jobs(ctx, layer, W, false, true, sage_first, &jobs);
  // the masked gradient, and where the aggregate gathers it in padded rows (layer_bwd_impl) those
  const int64_t rows = ctx->part.n_in + (dhalo ? (int64_t)expected_kept(ctx, p) : 0);
  const bool pad = dH_in && gather_stride(d_in, d_out) != d_out && d_out < d_in &&
                   (ctx->layer_kind == 0 || sage_first || tile_layer_bwd(ctx, layer, rows));
  BNS_TRY("relu_mask", relu_mask(ctx->part.n_in, d_out, dH_out, H_out, mask_scale_of(ctx), ctx->ws.G0,
                                 gather_stride(d_in, d_out), pad ? ctx->ws.G2 : nullptr, jobs, s));
  return layer_bwd_impl(ctx, layer, p, dZ, A_saved, H_in, W, dW, dH_in, dhalo, nullptr, false, nullptr, nullptr, 0.f, pad,
                        sage_first, nullptr, s);
}

// epoch_dev (nullable): the epoch index is read from there instead, and counted up by the last launch.
static bns_status train_step_impl(bns_ctx *ctx, uint64_t seed, uint32_t epoch, uint32_t *epoch_dev, double p,
                                  const float *X, const float *const *halo_h, const void *labels,
                                  float *const *W, float *const *dW, float *const *dhalo, float *loss, float lr,
                                  void *stream) {
  if (!ctx) return BNS_EINVAL;
  if (bad_p(p)) return fail(ctx, BNS_EINVAL, "p must lie in [0, 1]");
  if (!X || !labels || !W || !dW || !loss || (ctx->part.n_halo > 0 && !halo_h))
    return fail(ctx, BNS_EINVAL, "null pointer");
  const int L = ctx->n_layers, n_in = ctx->part.n_in;
  for (int l = 0; l < L; ++l)
    if (!W[l] || !dW[l] || (ctx->part.n_halo > 0 && !halo_h[l])) return fail(ctx, BNS_EINVAL, "null layer pointer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  Layout &w = ctx->ws;

  // the weights of up to kPackLayers layers are packed beside the sampling, those of deeper models before it
  PackJobs jobs;
  for (int l = L; l >= 1; --l) {
    add_pack_jobs(ctx, l, W[l - 1], true, l > 1, sage_gathers_first(ctx, l), &jobs);
    if (l > 1 && (l - 1) % kPackLayers == 0) {
      BNS_TRY("pack_weights", pack_weights(jobs, s));
      jobs = PackJobs{};
    }
  }
  if (timed(ctx, BNS_PHASE_SAMPLE)) {
    BNS_TRY("pack_weights", pack_weights(jobs, s));
    jobs = PackJobs{};
  }
  FirstLayer first{X, ctx->part.n_halo > 0 ? halo_h[0] : nullptr, W[0]};
  bns_status st = sample_and_build_impl(ctx, seed, epoch, epoch_dev, p, jobs, &first, s);
  if (st != BNS_OK) return st;

  const int C = ctx->dims[L];
  TnLoss loss_sum{w.loss_partials, 0, loss, epoch_dev};
  // where the last layer's backward pass gathers padded rows of dZ, the loss leaves them beside dZ
  const bool pad_last = pads_gradient(ctx, L, p, layer_plan(ctx, L, X) == BNS_LAYER_UPDATE_FIRST, L > 1);
  TileLoss last;
  last.labels = static_cast<const int32_t *>(labels);
  last.dZ = w.dZ[L];
  last.dZ_pad = pad_last ? w.G2 : nullptr;
  last.partials = w.loss_partials;
  last.ld = gather_stride(ctx->dims[L - 1], C);

  const float *H_prev = X;
  if (first.done) H_prev = w.H[1];
  for (int l = first.done ? 2 : 1; l <= L; ++l) {
    st = layer_fwd_impl(ctx, l, p, H_prev, ctx->part.n_halo > 0 ? halo_h[l - 1] : nullptr, W[l - 1], w.A[l],
                        w.H[l], l < L, layer_plan(ctx, l, X) == BNS_LAYER_UPDATE_FIRST, nullptr, l == L && ctx->loss_kind == 0 ? &last : nullptr, s);
    if (st != BNS_OK) return st;
    H_prev = w.H[l];
  }

  loss_sum.n = last.n_partials;
  if (loss_sum.n == 0) {
    PhaseTimer t(ctx, BNS_PHASE_LOSS, s);
    if (ctx->loss_kind == 0)
      BNS_TRY("loss_softmax_ce", loss_softmax_ce(n_in, C, w.H[L], last.labels, last.dZ, last.ld, last.dZ_pad,
                                                 last.partials, &loss_sum.n, s));
    else
      BNS_TRY("loss_sigmoid_bce", loss_sigmoid_bce(n_in, C, w.H[L], static_cast<const uint8_t *>(labels), last.dZ, last.ld, last.dZ_pad,
                                                   last.partials, &loss_sum.n, s));
  }

  // dZ[l] is the gradient w.r.t. the pre-activation of layer l; the backward pass of layer l writes
  // dZ[l-1], already masked by the activations of the layer below.  Every layer keeps its own buffer
  // (BNS_VIEW_DZ), so that each stage of the backward pass can be inspected with its exact inputs.
  const bool update_apart = lr > 0.f && timed(ctx, BNS_PHASE_SGD);
  TnBatch batch;
  for (int l = L; l >= 1; --l) {
    float *dh = (dhalo && l > 1) ? dhalo[l - 1] : nullptr;
    st = layer_bwd_impl(ctx, l, p, w.dZ[l], w.A[l], l > 1 ? w.H[l - 1] : X, W[l - 1], dW[l - 1],
                        l > 1 ? w.dZ[l - 1] : nullptr, dh,
                        l > 1 ? w.H[l - 1] : nullptr, layer_plan(ctx, l, X) == BNS_LAYER_UPDATE_FIRST,
                        ctx->part.n_halo > 0 ? halo_h[l - 1] : nullptr, W[l - 1], update_apart ? 0.f : lr, l == L && pad_last,
                        sage_gathers_first(ctx, l), &batch, s);
    if (st != BNS_OK) return st;
    if (l == 1 || batch.full()) {
      st = run_batch(ctx, &batch, l == 1 ? loss_sum : TnLoss{}, s);
      if (st != BNS_OK) return st;
    }
  }
  if (update_apart) {
    PhaseTimer t(ctx, BNS_PHASE_SGD, s);
    for (int l = 1; l <= L; ++l)
      BNS_TRY("sgd_update", sgd_update((int64_t)(ctx->layer_kind == 1 ? 2 : 1) * ctx->dims[l - 1] * ctx->dims[l], W[l - 1], dW[l - 1], lr, s));
  }
  return BNS_OK;
}

bns_status bns_train_step(bns_ctx *ctx, uint64_t seed, uint32_t epoch, double p, const float *X,
                          const float *const *halo_h, const void *labels, float *const *W, float *const *dW,
                          float *const *dhalo, float *loss, float lr, void *stream) {
  return train_step_impl(ctx, seed, epoch, nullptr, p, X, halo_h, labels, W, dW, dhalo, loss, lr, stream);
}

bns_status bns_graph_capture(bns_ctx *ctx, uint64_t seed, uint32_t first_epoch, double p, const float *X,
                             const float *const *halo_h, const void *labels, float *const *W, float *const *dW,
                             float *const *dhalo, float *loss, float lr, void *stream) {
  if (!ctx) return BNS_EINVAL;
  if (!stream) return fail(ctx, BNS_EINVAL, "graph capture needs a stream other than the null stream");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (ctx->graph_exec) { (void)hipGraphExecDestroy(ctx->graph_exec); ctx->graph_exec = nullptr; }
  uint32_t *epoch_dev = reinterpret_cast<uint32_t *>(ctx->ws.counters + 2);
  BNS_TRY("set_counter", set_counter(epoch_dev, first_epoch, s));
  BNS_TRY("hipStreamBeginCapture", hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
  // event brackets are not part of the graph: the phase timers are off between here and the end
  // of the capture, and there is no return in between
  const uint32_t saved_mask = ctx->prof.mask;
  ctx->prof.mask = 0;
  const int32_t *const drawn = ctx->drawn;
  const bool ws_built = ctx->ws_built;
  bns_status st = train_step_impl(ctx, seed, 0, epoch_dev, p, X, halo_h, labels, W, dW, dhalo, loss, lr, stream);
  ctx->cur_counted = false;  // recorded, not run
  ctx->drawn = drawn;
  ctx->ws_built = ws_built;
  hipGraph_t graph = nullptr;
  hipError_t e_end = hipStreamEndCapture(s, &graph);
  ctx->prof.mask = saved_mask;
  if (st != BNS_OK) { if (graph) (void)hipGraphDestroy(graph); return st; }
  if (e_end != hipSuccess) return hip_fail(ctx, "hipStreamEndCapture", e_end);
  hipError_t e_inst = hipGraphInstantiate(&ctx->graph_exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e_inst != hipSuccess) { ctx->graph_exec = nullptr; return hip_fail(ctx, "hipGraphInstantiate", e_inst); }
  return BNS_OK;
}

bns_status bns_graph_replay(bns_ctx *ctx, int32_t n_epochs, void *stream) {
  if (!ctx || n_epochs < 0) return BNS_EINVAL;
  if (!ctx->graph_exec) return fail(ctx, BNS_EINVAL, "bns_graph_capture has not been called");
  if (n_epochs > 0) {  // the keep bits are the replay's from here on, whose one-launch form does not count
    ctx->cur_counted = false;
    ctx->drawn = ctx->ws.remap;
    ctx->ws_built = true;
  }
  for (int i = 0; i < n_epochs; ++i)
    BNS_TRY("hipGraphLaunch", hipGraphLaunch(ctx->graph_exec, static_cast<hipStream_t>(stream)));
  return BNS_OK;
}

int32_t bns_layer_plan(const bns_ctx *ctx, int32_t layer) {
  if (!ctx || layer < 1 || layer >= (int32_t)ctx->dims.size()) return -1;
  return layer_plan(ctx, layer, ctx->cache_X);
}

bns_status bns_set_dropout(bns_ctx *ctx, double q) {
  if (!ctx) return BNS_EINVAL;
  if (!(q >= 0.0 && q < 1.0)) return fail(ctx, BNS_EINVAL, "dropout rate must lie in [0, 1)");
  ctx->drop_q = q;
  return BNS_OK;
}

bns_status bns_adam_update(float *W, const float *dW, float *m, float *v, int64_t n, float lr, float beta1,
                           float beta2, float eps, int32_t t, void *stream) {
  if (!W || !dW || !m || !v || n < 0 || t < 1) return BNS_EINVAL;
  if (!(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f)) return BNS_EINVAL;
  return adam_update(n, W, dW, m, v, lr, beta1, beta2, eps, t, static_cast<hipStream_t>(stream)) == hipSuccess
             ? BNS_OK
             : BNS_EHIP;
}

bns_status bns_cache_input_aggregate(bns_ctx *ctx, const float *X, void *stream) {
  if (!ctx) return BNS_EINVAL;
  ctx->cache_X = nullptr;
  if (!X) return BNS_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // C0[v,:] = sum over the inner neighbours u of v of d~_u^-1/2 X[u,:] (GCN layer) or of X[u,:]
  // without the self-loop (mean aggregator): static CSR, inner entries only, no row factor
  const bool sage = ctx->layer_kind == 1;
  SpmmRowPart part;
  part.row_take = ctx->ws.split.n_inner;
  part.skip_self = sage;
  BNS_TRY("spmm_fwd(cache)", spmm_fwd(ctx->ws.plan_f, ctx->part.n_in, ctx->dims[0], ctx->part.row_ptr0,
                                      ctx->part.col0, ctx->ws.w_fwd, ctx->ws.split.inner_ptr, nullptr, X, nullptr,
                                      ctx->ws.spmm_partials, ctx->ws.C0, part, false, false, s));
  ctx->cache_X = X;
  return BNS_OK;
}

bns_status bns_profile_enable(bns_ctx *ctx, uint32_t phase_mask, int32_t max_records) {
  if (!ctx || max_records < 0) return BNS_EINVAL;
  Profiler &pr = ctx->prof;
  pr.mask = phase_mask;
  pr.used = 0;
  while (pr.start.size() < (size_t)max_records) {
    hipEvent_t a, b;
    BNS_TRY("hipEventCreate", hipEventCreate(&a));
    pr.start.push_back(a);
    BNS_TRY("hipEventCreate", hipEventCreate(&b));
    pr.stop.push_back(b);
  }
  pr.phase.assign(pr.start.size(), 0);
  return BNS_OK;
}

bns_status bns_profile_read(bns_ctx *ctx, double *ms_per_phase, int32_t *records_per_phase) {
  if (!ctx || !ms_per_phase || !records_per_phase) return BNS_EINVAL;
  Profiler &pr = ctx->prof;
  for (int i = 0; i < BNS_PHASE_COUNT; ++i) { ms_per_phase[i] = 0.0; records_per_phase[i] = 0; }
  for (size_t k = 0; k < pr.used; ++k) {
    BNS_TRY("hipEventSynchronize", hipEventSynchronize(pr.stop[k]));
    float ms = 0.f;
    BNS_TRY("hipEventElapsedTime", hipEventElapsedTime(&ms, pr.start[k], pr.stop[k]));
    ms_per_phase[pr.phase[k]] += ms;
    records_per_phase[pr.phase[k]] += 1;
  }
  pr.used = 0;
  return BNS_OK;
}

bns_status bns_ws_view(const bns_ctx *ctx, bns_view which, int32_t layer, void **dev_ptr, size_t *bytes) {
  if (!ctx || !dev_ptr || !bytes) return BNS_EINVAL;
  const Layout &w = ctx->ws;
  const size_t n_in = ctx->part.n_in, B = ctx->part.n_halo, nnz0 = ctx->part.nnz0;
  switch (which) {
    case BNS_VIEW_KEPT_IDS: *dev_ptr = w.kept_ids; *bytes = 4 * B; break;
    case BNS_VIEW_REMAP: *dev_ptr = w.remap; *bytes = 4 * B; break;
    case BNS_VIEW_N_KEPT: *dev_ptr = w.counters; *bytes = 4; break;
    case BNS_VIEW_ROW_PTR: *dev_ptr = w.row_ptr; *bytes = 4 * (n_in + 1); break;
    case BNS_VIEW_COL_IDX: *dev_ptr = w.col_idx; *bytes = 4 * nnz0; break;
    case BNS_VIEW_T_ROW_PTR: *dev_ptr = w.t_row_ptr; *bytes = 4 * (n_in + B + 1); break;
    case BNS_VIEW_T_COL_IDX: *dev_ptr = w.t_col_idx; *bytes = 4 * nnz0; break;
    case BNS_VIEW_NNZ: *dev_ptr = w.counters + 1; *bytes = 4; break;
    case BNS_VIEW_A:
    case BNS_VIEW_H:
    case BNS_VIEW_DZ:
      if (layer < 1 || layer > ctx->n_layers) return BNS_EINVAL;
      if (which == BNS_VIEW_A) { *dev_ptr = w.A[layer]; *bytes = 4 * n_in * (size_t)ctx->dims[layer - 1]; }
      else if (which == BNS_VIEW_H) { *dev_ptr = w.H[layer]; *bytes = 4 * n_in * (size_t)ctx->dims[layer]; }
      else { *dev_ptr = w.dZ[layer]; *bytes = 4 * n_in * (size_t)ctx->dims[layer]; }
      break;
    default: return BNS_EINVAL;
  }
  return BNS_OK;
}

}  // extern "C"
