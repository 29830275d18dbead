// Selection step, subgraph step and the first layer's forward pass of a small partition in one launch.
//
// The first layer waits for the subgraph, and a launch is 2.5 us before its first read.  But what it needs of the subgraph are its rows' entries,
// and these follow from the static lists and the draws of the boundary nodes in them, which are a function of the node: a wavefront forms its row's
// entries itself, the inner ones and then the boundary nodes that are kept, in batches of 64 as the sampled row has them, and so the
// aggregate has the order of sums, and the bits, of the launch on the finished subgraph.  Workgroup 0 writes the subgraph for the later launches
// meanwhile, others pack the weights.  What it costs is a draw per boundary entry and a read that depends on the entry's list: workgroup 0 takes 5.4 us by
// itself, all of it 6.4, the layer by itself 5.0 (500 rows, 64 -> 16; step 24.6 -> 21.0).
#include "pack_device.hpp"
#include "small_device.hpp"
#include "tile_device.hpp"

namespace bns {

namespace {

constexpr int kTilesPerGroup = kSmallThreads / (kTileWaves * kWave);

struct FirstArgs {
  SmallArgs small;
  TileArgs tile;       // row_ptr, col_idx and halo_rec of the subgraph are not read
  bool skip_inner;     // the inner entries' sum is tile.sp.init
  int32_t pack_groups;
  PackJobs pack;
};

struct Entry {
  int32_t from;  // inner node, or ~boundary node
  float w;
};

// The lanes' writes to their wavefront's list are seen by all of its lanes.
__device__ __forceinline__ void list_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The rows row0 .. + rows of the aggregate out of the static lists; wid: of the tile's wavefronts.
template <int LPR, typename Put>
__device__ __forceinline__ void gather_drawn(const FirstArgs &f, int wid, Entry (&list)[2 * kWave], uint32_t epoch, int row0, int rows, Put put) {
  const SpmmArgs &a = f.tile.sp;
  const SmallArgs &s = f.small;
  const int lane = lane_id(), g = lane / LPR, sl = lane % LPR, d = a.d, nvec = d / 4;
  for (int r = wid; r < rows; r += kTileWaves) {
    const int row = row0 + r;
    const int2 in = scalar_load_pair(s.sp.inner_ptr, row), bd = scalar_load_pair(s.sp.bd_ptr, row);
    // what the first batch of either kind reads, all at once
    int c = 0, b = 0;
    float w = 1.f, dis = 1.f;
    int64_t gid = 0;
    const int n_in = f.skip_inner ? 0 : in.y - in.x, n_bd = bd.y - bd.x;
    auto ask_inner = [&](int at) {
      if (at + lane < n_in) {
        c = s.sp.in_col[in.x + at + lane];
        if (a.w_in) w = a.w_in[in.x + at + lane];
      }
    };
    auto ask_boundary = [&](int at) {
      if (at + lane < n_bd) {
        b = s.sp.bd_b[bd.x + at + lane];
        gid = s.halo_gid[b];
        if (s.dis_halo) dis = s.dis_halo[b];
      }
    };
    ask_inner(0);
    ask_boundary(0);
    float acc[1][4] = {};
    int have = 0, at_in = 0, at_bd = 0;  // entries in the list; those taken of either kind
    while (have > 0 || at_in < n_in || at_bd < n_bd) {
      if (at_in < n_in) {  // (the list is empty)
        have = min(kWave, n_in - at_in);
        if (lane < have) list[lane] = Entry{c, w};
        at_in += have;
        ask_inner(at_in);
      } else if (at_bd < n_bd) {
        bool keep = false;
        if (at_bd + lane < n_bd) {
          uint32_t c0 = (uint32_t)gid, c1 = (uint32_t)((uint64_t)gid >> 32), c2 = epoch, c3 = s.part_id;
          philox4x32_10(c0, c1, c2, c3, s.k0, s.k1);
          keep = (uint64_t)c0 < s.threshold;
        }
        const unsigned long long kept = __ballot(keep);
        if (keep) list[have + __popcll(kept & ((1ull << lane) - 1ull))] = Entry{~b, s.dis_halo ? s.s_halo * dis : s.s_halo};
        have += __popcll(kept);
        at_bd = min(n_bd, at_bd + kWave);
        ask_boundary(at_bd);
      }
      if (have < kWave && (at_in < n_in || at_bd < n_bd)) continue;
      list_sync();
      const int cnt = min(have, kWave);
      unsigned long long p = 0;
      float we = 0.f;
      constexpr bool DPP = dpp_gather(1, LPR);
      const int mine = batch_entry<LPR, DPP>();
      if (mine < cnt) {
        const Entry e = list[mine];
        p = (unsigned long long)(e.from >= 0 ? a.src0 + (size_t)e.from * d : a.src1 + (size_t)~e.from * d);
        we = a.skip_self && e.from == row ? 0.f : e.w;
      }
      gather_batch<4, 1, LPR, DPP>(p, we, cnt, nvec, acc);
      have -= cnt;
      if (have > 0) {
        const Entry e = list[kWave + lane];
        list_sync();
        if (lane < have) list[lane] = e;
      }
    }
    fold_groups<4, 1, LPR>(acc);
    if (g == 0) put(row, sl, acc);
  }
}

template <int LPR, int VW, bool SAGE, bool LARGE>
__global__ void __launch_bounds__(kSmallThreads) first_layer_kernel(const FirstArgs f) {
  if (blockIdx.x == 0) {
    constexpr int NB = LARGE ? kSmallMaxHalo / kSmallThreads : 1, NE = LARGE ? kSmallMaxBoundaryEntries / kSmallThreads : 1;
    sample_and_build<NB, NE>(f.small);
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = (int)blockIdx.x - 1 - f.pack_groups;
  if (group < 0) {
    pack_unit(f.pack, ((int)blockIdx.x - 1) * (kSmallThreads / kWave) + wave);
    return;
  }
  __shared__ __attribute__((aligned(16))) float As[kTilesPerGroup][SAGE ? 2 : 1][kTileRows * kTileLd];
  __shared__ Entry lists[kSmallThreads / kWave][2 * kWave];
  const int part = wave / kTileWaves;
  const uint32_t epoch = f.small.epoch_dev ? *f.small.epoch_dev : f.small.epoch;
  tile_layer<LPR, VW, SAGE, false>(f.tile, group * kTilesPerGroup + part, threadIdx.x % (kTileWaves * kWave), As[part], [&](int row0, int rows, auto put) {
    gather_drawn<LPR>(f, wave % kTileWaves, lists[wave], epoch, row0, rows, put);
  });
}

}  // namespace

hipError_t sample_build_first(const SmallArgs &small, const PackJobs &pack, int32_t d_in, int32_t d_out, const float *w_in, const float *row_scale,
                              const float *H_in, const float *halo_h, float *A, const float *cached, const float *W, float *H_out,
                              bool relu, const Dropout &drop, bool sage, bool concat, const SegPlan &plan, hipStream_t s) {
  if (!tile_layer_supported(plan, d_in, d_out) || plan.n_multi > 0 || small.n_halo > kSmallMaxHalo || small.e_bd > kSmallMaxBoundaryEntries)
    return hipErrorInvalidValue;
  FirstArgs f;
  f.small = small;
  SpmmRowPart part;
  part.init = cached;
  part.skip_self = sage;
  f.tile.sp = spmm_fwd_args(plan, small.n_in, d_in, nullptr, nullptr, w_in, nullptr, row_scale, H_in, halo_h, nullptr, A, part);
  f.tile.W = W;
  f.tile.H_self = sage ? H_in : nullptr;
  f.tile.H_out = H_out;
  f.tile.d_out = d_out;
  f.tile.rows = tile_rows(small.n_in);
  f.tile.relu = relu;
  f.tile.concat = concat;
  f.tile.drop = drop;
  f.skip_inner = cached != nullptr;
  f.pack = pack;
  f.pack_groups = (pack.units + kSmallThreads / kWave - 1) / (kSmallThreads / kWave);
  const int tiles = (small.n_in + f.tile.rows - 1) / f.tile.rows;
  const unsigned blocks = (unsigned)(1 + f.pack_groups + (tiles + kTilesPerGroup - 1) / kTilesPerGroup);
  const bool large = small.n_halo > kSmallThreads || small.e_bd > kSmallThreads;
#define BNS_FIRST_KIND(LPR, VW, SAGE)                                                                            \
  do {                                                                                                           \
    if (large) first_layer_kernel<LPR, VW, SAGE, true><<<blocks, kSmallThreads, 0, s>>>(f);                     \
    else first_layer_kernel<LPR, VW, SAGE, false><<<blocks, kSmallThreads, 0, s>>>(f);                          \
  } while (0)
#define BNS_FIRST(LPR, VW)                            \
  do {                                                \
    if (sage) BNS_FIRST_KIND(LPR, VW, true);          \
    else BNS_FIRST_KIND(LPR, VW, false);              \
  } while (0)
  const bool wide = d_out > 16 * kTileWaves;
  if (d_in > 64) BNS_FIRST(32, 1);
  else if (d_in > 32) { if (wide) BNS_FIRST(16, 2); else BNS_FIRST(16, 1); }
  else if (d_in > 16) { if (wide) BNS_FIRST(8, 2); else BNS_FIRST(8, 1); }
  else { if (wide) BNS_FIRST(4, 2); else BNS_FIRST(4, 1); }
#undef BNS_FIRST
#undef BNS_FIRST_KIND
  return hipGetLastError();
}

}  // namespace bns
