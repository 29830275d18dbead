// Sparse aggregate (Eq. 1 in the sampled matrix form of Appendix A) and its transpose.
//
// Work unit: one 64-lane wavefront owns one SEGMENT of an output row, at most kSegLen
// neighbours.  Power-law graphs put a large share of all edges into a few very long rows; cutting
// every row into bounded segments keeps the wavefronts balanced.  A row with one segment is
// finished by its wavefront; a row with several gets one partial sum per segment, and these are added in ascending order by whoever
// launch_spmm_vec says: the workgroup that owns the row, the wavefront that finishes its last segment, or a second small kernel.  No atomics on values
// anywhere: the backward pass walks the transposed pattern, and every output element is produced in a fixed order.
//
// Inside a segment the lanes span the feature dimension with VEC-wide loads, so every neighbour
// row is read as one contiguous, coalesced piece (four floats to a lane, whatever the width, from 9 on).  When a feature row needs fewer than 64 lanes
// (LPR = lanes per row < 64) the wavefront walks 64/LPR neighbours at once and folds the partial
// sums at the end.  Column indices and their weights are fetched 64 at a time, one per lane,
// and handed to the loop by cross-lane reads, four neighbours in flight per step.
#include <algorithm>

#include "pack_device.hpp"
#include "spmm_device.hpp"

namespace bns {

// Where launch_spmm_vec says so: a segment's partial sum is on its way, and the wavefront that is the last of its row (and slice) to get here adds up the row, in
// ascending order of the segments.  The partial sums are written and read at the agent's scope (shared_store, shared_load), past the caches of one XCD, so that
// nothing has to be flushed; on the one side the store has ended before the segment is counted, on the other no partial sum is asked for before the count has
// come back and says that all have.  With plain loads, or loads asked for earlier, the last wavefront would add up what its own L2 had held before.
template <int VEC, int MAXCH, int LPR, bool NARROW, bool RAGGED>
__device__ __forceinline__ void finish_long_row(int row, int d_off) {
  using V = typename Vec<VEC, RAGGED>::T;
  ArgBlock &a = unit_args();
  if (a.plan.arrived == nullptr) return;  // a launch behind this one adds them up
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  int lane = lane_id();
  asm volatile("" : "+v"(lane));  // (found again rather than kept in registers beside the gather)
  const int slot0 = scalar_load(a.plan.part_ptr, row);
  const int2 seg = scalar_load_pair(a.plan.seg_ptr, row);
  const int nseg = seg.y - seg.x;
  int32_t *const count = a.plan.arrived + 4 * slot0 + d_off / a.head.d_slice;
  int before = 0;
  if (lane == 0) before = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (__builtin_amdgcn_readfirstlane(before) != nseg - 1) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");  // (no instruction: the loads below stay below)
  if (lane == 0) __hip_atomic_store(count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
  if (lane >= LPR) return;
  const int width = RAGGED ? min(a.head.d_slice, a.d - d_off) : a.head.d_slice, nvec = (width + (RAGGED ? VEC - 1 : 0)) / VEC;
  const float *const part = a.partials + (size_t)slot0 * a.d + d_off;
  float acc[MAXCH][VEC] = {};
  constexpr int CU = MAXCH == 1 ? 8 : 4;  // partial sums fetched together
  for (int s0 = 0; s0 < nseg; s0 += CU) {
    V x[CU][MAXCH];
#pragma unroll
    for (int t = 0; t < CU; ++t)
#pragma unroll
      for (int c = 0; c < MAXCH; ++c)  // (a piece past the end of the row, and a segment past the last one, are the last one again)
        x[t][c] = shared_load<VEC, V>(part + (size_t)min(s0 + t, nseg - 1) * a.d, piece_at<VEC, RAGGED>(min(c * kWave + lane, nvec - 1), width));
    asm volatile("" ::: "memory");  // none of them moves behind a condition below, where it would be waited for before the next
#pragma unroll
    for (int t = 0; t < CU; ++t) {
      const bool there = s0 + t < nseg;
#pragma unroll
      for (int c = 0; c < MAXCH; ++c)
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          const float sum = acc[c][i] + reinterpret_cast<const float *>(&x[t][c])[i];
          acc[c][i] = there ? sum : acc[c][i];
        }
    }
  }
  finish_row<VEC, MAXCH, NARROW, RAGGED>(unit_args(), row, lane, nvec, d_off, acc, width);
}

// BLOCK: workgroups of kBlockWaves wavefronts; the first plan.n_multi of them own a multi-segment row each, one
// wavefront per segment, and add the partial sums in LDS (same order as finish_long_row, same bits).  In front of the
// others are head.n_block_rows workgroups, n_multi rounded up to whole groups; those past n_multi have nothing to do.
constexpr int kBlockWaves = 8;
template <int VEC, int MAXCH, int LPR, bool NARROW = false, bool BLOCK = false, bool RAGGED = false, bool SHORT = false>
__global__ void __launch_bounds__(BLOCK ? kBlockWaves * kWave : 256, MAXCH == 1 ? 8 : 1) spmm_kernel(const SpmmArgs) {
  using V = typename Vec<VEC, RAGGED>::T;
  constexpr int kCut = RAGGED ? VEC - 1 : 0;  // (a last piece that is not whole)
  constexpr int kWaves = BLOCK ? kBlockWaves : 4;
  const int lane = lane_id();
  const int g = lane / LPR, sl = lane % LPR;
  int bid = blockIdx.x, d_off = 0;
  const SpmmArgs::Head start = unit_head();
  if (const int ls = start.log2_slices) {  // gridDim.x is a multiple of 8
    const int x = bid & 7;
    bid = ((bid >> 3) << (3 - ls)) + (x >> ls);
    d_off = ((x + (int)__umulhi(bid, start.turn_share)) & ((1 << ls) - 1)) * start.d_slice;
  }
  // (the unit is the same for the whole wavefront, so that its bounds come through the scalar cache)
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (BLOCK) {
    const int n_rows = start.n_block_rows;
    if (bid < n_rows) {
      ArgBlock &a = unit_args();
      extern __shared__ __attribute__((aligned(16))) float block_part[];
      const int ds = start.d_slice, width = RAGGED ? min(ds, a.d - d_off) : ds, nvec = (width + kCut) / VEC;
      const int n_multi = a.plan.n_multi;  // (asked for beside the row, which the others wait for)
      const int row = scalar_load(a.plan.mrow, min(bid, n_multi - 1));
      if (bid >= n_multi) return;
      const int2 ee = scalar_load_pair(a.row_ptr, row);
      int e0 = ee.x, e1 = ee.y;
      const InnerWeights iw = inner_weights(a, row, e0, e1);
      if (a.row_skip) e0 += scalar_load(a.row_skip, row);
      if (a.row_take) e1 = e0 + scalar_load(a.row_take, row);
      const int2 seg = scalar_load_pair(a.plan.seg_ptr, row);
      const int nseg = seg.y - seg.x;  // <= kWaves
      const int chunk = (e1 - e0 + nseg - 1) / nseg;
      float acc[MAXCH][VEC];
      if (wid < nseg) {
        const int b = min(e1, e0 + wid * chunk);
        gather_segment<VEC, MAXCH, LPR, RAGGED>(a, row, iw, b, min(e1, b + chunk), d_off, nvec, acc, width);
        if (g == 0) {
#pragma unroll
          for (int c = 0; c < MAXCH; ++c)
            if (c * kWave + sl < nvec)
#pragma unroll
              for (int i = 0; i < VEC; ++i) block_part[wid * ds + piece_at<VEC, RAGGED>(c * kWave + sl, width) + i] = acc[c][i];
        }
      }
      __syncthreads();
      if (wid != 0) return;
#pragma unroll
      for (int c = 0; c < MAXCH; ++c)
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[c][i] = 0.f;
      for (int s = 0; s < nseg; ++s)
#pragma unroll
        for (int c = 0; c < MAXCH; ++c)
          if (c * kWave + lane < nvec)
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[c][i] += block_part[s * ds + piece_at<VEC, RAGGED>(c * kWave + lane, width) + i];
      finish_row<VEC, MAXCH, NARROW, RAGGED>(unit_args(), row, lane, nvec, d_off, acc, width);
      return;
    }
    bid -= n_rows;
  }
  // A static unit per wavefront, and the kept boundary rows (their count is on the device): in workgroups of their own,
  // extra_share in 2^32 of the groups of 8, or on all wavefronts after their units.
  int unit = bid * kWaves + wid, end = start.n_units, step = start.extra_step;
  if (const unsigned share = start.extra_share) {
    const int group_bits = 3 - start.log2_slices, in_group = bid & ((1 << group_bits) - 1);
    int group = bid >> group_bits;
    if ((group | 31) < start.n_groups) group = (group & ~31) | (int)(__brev(group) >> 27);
    const int before = __umulhi(group, share);  // such groups before this one
    if ((int)__umulhi(group + 1, share) != before) {
      unit = end + ((before << group_bits) + in_group) * kWaves + wid;
      end += scalar_load(unit_args().n_extra_dev, 0);
    } else {
      unit = (((group - before) << group_bits) + in_group) * kWaves + wid;
      step = end;
    }
  } else if (const int32_t *n = unit_args().n_extra_dev) {
    const int extra = scalar_load(n, 0);
    end += SHORT ? (extra + kShortRows - 1) / kShortRows : extra;
  }
  for (int next = 0; unit < end; unit += SHORT ? 0 : step) {  // SHORT: the kept boundary rows are units of kShortRows, `next` the one to go on with
    ArgBlock &a = unit_args();
    const int width = RAGGED ? min(a.head.d_slice, a.d - d_off) : a.head.d_slice, nvec = (width + kCut) / VEC;
    int row = a.n_split + (unit - a.head.n_units), slot = -1;
    if (unit < a.head.n_units) {
      const int2 u = scalar_load(a.units, unit);
      row = u.x;
      slot = u.y;
      if (SHORT) unit += step;
    } else if constexpr (SHORT) {
      const int r0 = (unit - a.head.n_units) * kShortRows, n = min(kShortRows, scalar_load(a.n_extra_dev, 0) - r0);
      row = a.n_split + r0;
      if (next == 0 && scalar_load(a.row_ptr, row + n) - scalar_load(a.row_ptr, row) <= kWave) {
        short_rows<VEC, LPR, NARROW, RAGGED>(a, r0, n, d_off, nvec, width);
        unit += step;
        continue;
      }
      row += next;  // one after another
      if (++next == n) {
        next = 0;
        unit += step;
      }
    }
    const int2 ee = scalar_load_pair(a.row_ptr, row);
    int e0 = ee.x, e1 = ee.y;
    const InnerWeights iw = inner_weights(a, row, e0, e1);
    if (row < a.n_split) {
      if (a.row_skip) e0 += scalar_load(a.row_skip, row);
      if (a.row_take) e1 = e0 + scalar_load(a.row_take, row);
    }
    if (slot >= 0) {  // this wavefront's slice of the row as it is in this epoch
      const int seg = slot - scalar_load(a.plan.part_ptr, row);
      const int nseg = scalar_load(a.plan.seg_ptr, row + 1) - scalar_load(a.plan.seg_ptr, row);
      const int chunk = (e1 - e0 + nseg - 1) / nseg;
      e0 = min(e1, e0 + seg * chunk);
      e1 = min(e1, e0 + chunk);
    }

    float acc[MAXCH][VEC];
    gather_segment<VEC, MAXCH, LPR, RAGGED>(a, row, iw, e0, e1, d_off, nvec, acc, width);

    ArgBlock &b = unit_args();
    if (g != 0) {
      // only the first lane group holds the folded sums
    } else if (slot < 0) {
      finish_row<VEC, MAXCH, NARROW, RAGGED>(b, row, sl, nvec, d_off, acc, width);
    } else {
      float *part = b.partials + (size_t)slot * b.d + d_off;
#pragma unroll
      for (int c = 0; c < MAXCH; ++c) {
        const int iv = c * kWave + sl;
        if (iv < nvec) {
          V o;
          float *po = reinterpret_cast<float *>(&o);
#pragma unroll
          for (int i = 0; i < VEC; ++i) po[i] = acc[c][i];
          if (b.plan.arrived) shared_store<VEC>(part, piece_at<VEC, RAGGED>(iv, width), o);
          else *piece_of<VEC, RAGGED>(part, iv, width) = o;
        }
      }
    }
    if (!BLOCK && slot >= 0) finish_long_row<VEC, MAXCH, LPR, NARROW, RAGGED>(row, d_off);
  }
}

// The segments of the long rows ahead of a one-kernel layer of 128 floats, in two slices over the XCDs.  Whole rows of 128 go to 32 lanes each, so that a
// segment has two running sums, and a launch must not give it others: sums in another order switch hidden units within rounding of
// zero.  64 lanes on a slice would make four sums (of 64 floats) or eight (of 32).  So a wavefront takes two segments, which follow each other
// in the columns' order: 32 lanes to a segment, 16 to an entry, four entries to a load.  The next batch's columns and
// weights are asked for before a batch is gathered: there is one chain of reads for two segments.
// Us, whole rows / so / with eight sums (not kept): 306250 rows of 45 entries 210 / 182 / 159, 578125 of 21 212 / 200 / 182, 100000 of 92 130 / 117 / 114, of
// 196 309 / 277 / 275, 250000 of 20 74 / 71 / 59; with 9 % of boundary entries, which are looked up in the kept nodes' records in every slice, 306250 of 50
// 259 / 245 / 227, with 24 % of 59 354 / 343, with 26 % 578125 of 28 349 / 358.  One segment to a wavefront, two floats to a lane, the first four 183, 194, 135,
// 332; four segments in slices of 32 floats 176, 207, 133, 310.
constexpr int kLongPerWave = 2;
template <int T0, typename F>
__device__ __forceinline__ void eight_steps(F f) {
  f(std::integral_constant<int, T0>{}); f(std::integral_constant<int, T0 + 1>{}); f(std::integral_constant<int, T0 + 2>{}); f(std::integral_constant<int, T0 + 3>{});
  f(std::integral_constant<int, T0 + 4>{}); f(std::integral_constant<int, T0 + 5>{}); f(std::integral_constant<int, T0 + 6>{}); f(std::integral_constant<int, T0 + 7>{});
}
__global__ void __launch_bounds__(256, 8) spmm_long_kernel(const SpmmArgs) {
  constexpr int VEC = 4, kLanes = kWave / kLongPerWave, EP = 2, kSteps = kLanes / EP;  // lanes of a segment, entries to a step, steps of a batch
  const SpmmArgs::Head start = unit_head();
  const int ls = start.log2_slices, x = blockIdx.x & 7;
  const int bid = ((blockIdx.x >> 3) << (3 - ls)) + (x >> ls);
  const int d_off = ((x + (int)__umulhi(bid, start.turn_share)) & ((1 << ls) - 1)) * start.d_slice;
  const int lane = lane_id(), ln = lane % kLanes, g = ln / kSteps, sl = lane % kSteps;
  const int first = (bid * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kLongPerWave, unit = first + lane / kLanes;
  ArgBlock &a = unit_args();
  const int2 u = a.units[min(unit, start.n_units - 1)];
  const int row = u.x;
  int e0 = a.row_ptr[row], e1 = a.row_ptr[row + 1], w_at = 0, w_end = e0;  // the weight of entry e < w_end is w_in[e + w_at]
  if (a.w_in) {
    const int w0 = a.w_ptr[row];
    w_at = w0 - e0;
    w_end = e0 + (a.w_ptr[row + 1] - w0);
  }
  const int s0 = a.plan.seg_ptr[row], nseg = a.plan.seg_ptr[row + 1] - s0, seg = u.y - a.plan.part_ptr[row];
  if (a.row_skip) e0 += a.row_skip[row];
  if (a.row_take) e1 = e0 + a.row_take[row];
  const int chunk = (e1 - e0 + nseg - 1) / nseg;
  e0 = min(e1, e0 + seg * chunk);
  e1 = unit < start.n_units ? min(e1, e0 + chunk) : e0;
  float acc[1][VEC] = {};
  int c_next = 0;
  float w_next = 0.f;
  auto ask = [&](int e, int n) {
    if (ln < n) {
      if (e < w_end) w_next = a.w_in[e + w_at];
      c_next = a.col_idx[e];
    }
  };
  int e = e0 + ln, cnt = e1 - e0;  // (cnt: 0 and less where the other segment is the longer one)
  ask(e, cnt);
  for (; __any(cnt > 0); cnt -= kLanes) {
    // step t takes entries EP t + g of the batch; lane t of the sixteen holds that one (fetched in their own order: batch_entry)
    int l = lane_id();
    asm volatile("" : "+v"(l));  // (found again rather than kept in registers beside the gather)
    const int mine = (l % kSteps) * EP + l / kSteps % EP, from = l / kLanes * kLanes + mine;
    const int c = __shfl(c_next, from, kWave);
    const float w_e = __shfl(w_next, from, kWave);
    w_next = 0.f;
    e += kLanes;
    ask(e, cnt - kLanes);
    unsigned long long p_l = 0;
    float w_l = 0.f;
    if (mine < cnt) entry_source(a, row, c, d_off, p_l, w_l, [&] { return a.w_in ? w_e : 1.f; });
    const unsigned lo_l = (unsigned)p_l, hi_l = (unsigned)(p_l >> 32), w_u = __float_as_uint(w_l);
    auto steps = [&](auto whole, auto t0) {
      constexpr int T0 = decltype(t0)::value;
      Vec<VEC>::T v[8];
      eight_steps<T0>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        const unsigned lo = row_bcast<t>(lo_l), hi = row_bcast<t>(hi_l);
        v[t - T0] = Vec<VEC>::T{};
        if (decltype(whole)::value || t * EP + g < cnt) v[t - T0] = load_row_piece<VEC, false>(hi, lo, sl * VEC);
      });
      eight_steps<T0>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        vec_fma<VEC>(acc[0], __uint_as_float(row_bcast<t>(w_u)), reinterpret_cast<const float *>(&v[t - T0]));
      });
    };
    const std::integral_constant<int, 0> t0;
    const std::integral_constant<int, 8> t8;
    if (__all(cnt >= 8 * EP)) steps(std::true_type{}, t0);
    else steps(std::false_type{}, t0);
    if (__all(cnt >= 16 * EP)) steps(std::true_type{}, t8);
    else if (__any(cnt > 8 * EP)) steps(std::false_type{}, t8);
  }
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[0][i] = lane_pair_sum(acc[0][i], kSteps);
  if (g != 0) return;
  ArgBlock &b = unit_args();
  int at = lane_id();
  asm volatile("" : "+v"(at));
  const int done = first + at / kLanes;
  if (done >= start.n_units) return;
  Vec<VEC>::T o;
#pragma unroll
  for (int i = 0; i < VEC; ++i) reinterpret_cast<float *>(&o)[i] = acc[0][i];
  reinterpret_cast<Vec<VEC>::T *>(b.partials + (size_t)b.units[done].y * b.d + d_off)[sl] = o;
}

// Rows cut into several segments: add the partial sums in ascending segment order.
template <int VEC, int MAXCH, bool NARROW = false, bool RAGGED = false>
__global__ void __launch_bounds__(256) spmm_combine_kernel(const SpmmArgs a) {
  using V = typename Vec<VEC, RAGGED>::T;
  const int lane = lane_id();
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= a.plan.n_multi) return;
  const int row = a.plan.mrow[j];
  const int nseg = a.plan.seg_ptr[row + 1] - a.plan.seg_ptr[row];
  const int d = a.d, nvec = (d + (RAGGED ? VEC - 1 : 0)) / VEC;
  const float *part = a.partials + (size_t)a.plan.part_ptr[row] * d;
  float acc[MAXCH][VEC];
#pragma unroll
  for (int c = 0; c < MAXCH; ++c)
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[c][i] = 0.f;
  constexpr int CU = 8;  // partial vectors fetched together; they are still added in ascending order
  for (int s0 = 0; s0 < nseg; s0 += CU) {
    V x[CU][MAXCH];
#pragma unroll
    for (int t = 0; t < CU; ++t) {
      const float *ps = part + (size_t)(s0 + t) * d;
#pragma unroll
      for (int c = 0; c < MAXCH; ++c) {
        const int iv = c * kWave + lane;
        x[t][c] = (s0 + t < nseg && iv < nvec) ? *piece_of<VEC, RAGGED>(ps, iv, d) : V{};
      }
    }
#pragma unroll
    for (int t = 0; t < CU; ++t)
#pragma unroll
      for (int c = 0; c < MAXCH; ++c) {
        const float *px = reinterpret_cast<const float *>(&x[t][c]);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[c][i] += px[i];
      }
  }
  finish_row<VEC, MAXCH, NARROW, RAGGED>(a, row, lane, nvec, 0, acc, d);
}

constexpr int kByLastMaxParts = 45056, kByLastMaxSegments = 64, kResidentWaves = 8192;  // of by_last below
template <int VEC, bool RAGGED>
static hipError_t launch_spmm_vec(const SpmmArgs &a_in, int64_t extra_rows, bool multi_only, int32_t avg_len, bool transposed, hipStream_t s) {
  SpmmArgs a = a_in;
  // multi_only: the segments of the multi-segment rows, which come first
  const int64_t n_units = a.head.n_units = multi_only ? a.plan.n_part : a.plan.n_seg;
  a.units = a.plan.order;
  // Wide rows are cut into slices of 128 floats (64 where rows are long enough to keep a
  // wavefront busy with a quarter of its lanes per neighbour): narrower slices lose more to the repeated index walk than
  // the L2 gains.  In the transposed pass that line is counted in entries per row of the whole launch, the short rows of the
  // boundary nodes among them, and depends on what the narrower slices bring (slices of 128 -> of 64, us):
  //   more wavefronts, where those of 128 do not fill the chip: 4600 rows of 128 floats with 20.4 entries 19 -> 17, 2500 of
  //     256 with 26.9 14 -> 13;
  //   room in the L2 for rows that do not fit it: 2 slices instead of 1 from 19 entries on (60000 rows with 17.6 74 -> 77,
  //     with 21.3 87 -> 80; 300000 with 21.3 508 -> 474; 886000 with 14.5 853 -> 991, with 19.6 1108 -> 1132), more slices from
  //     24 on (60000 rows of 256 with 21.3 150 -> 153, with 26 182 -> 165; of 512 277 -> 289, 332 -> 307);
  //   neither, in between: from 32 on (9000 rows of 512 with 26.9 entries 41 -> 48, 16000 70 -> 81; 16000 of 256 with 56.6 70 -> 68).
  // A forward row keeps the order of its sum, and so its slices (from 64 entries on): see spmm_long_kernel.
  int ls = 0;
  if (VEC == 4 && !multi_only) {
    auto slices = [&](int target) {
      int l = 0;
      while (l < 3 && (a.d >> (l + 1)) >= target && (RAGGED || a.d % (VEC << (l + 1)) == 0)) ++l;
      return l;
    };
    ls = slices(128);
    int from = 64;
    if (transposed)
      from = (n_units << ls) <= 8192 ? 19 : n_units < 24576 ? 32 : ls == 0 ? 19 : 24;
    if (avg_len >= from) ls = slices(64);
  }
  const bool by_two = VEC == 4 && !RAGGED && multi_only && a.d == 128;  // spmm_long_kernel: the one width of whole lines in two slices (68 to 128 there are)
  if (by_two) ls = 1;
  a.head.log2_slices = ls;
  a.head.d_slice = RAGGED && ls > 0 ? ((a.d + (1 << ls) - 1) / (1 << ls) + 3) / 4 * 4 : a.d >> ls;  // (the last one of a ragged row is narrower)
  // The pass over the partial sums is a launch: 4.7 to 5.5 us for 1300 segments of 89625 rows, 7.2 to 8.2 for 23200 of 306250, 8 to 13 for 40500 of 29125, 18 for
  // 16900 of 578125, 169 of them in one row.  Where the longest row has few segments, a workgroup per such row saves it; its workgroups of
  // eight wavefronts wait for their longest row, which costs more where wavefronts are many and run at the rate of the LDS or vector pipes, i.e. in slices of 33 to 64 floats: those cross at about 20000 units (12000
  // rows in 2 slices 29.2 us, in blocks 30.2; 20000 in 2 38, 43; in 4 67, 80; 30000 whole rows 26.4, 27.6), rows of 9 to 32
  // floats at 50000 to 100000, wider ones not up to 100000 (128 floats: 12000 rows 36 and 33 us, 100000 155 and 149).
  const bool narrow_slice = a.head.d_slice > 32 && a.head.d_slice <= 64;
  const bool block_rows = !multi_only && a.plan.n_multi > 0 && a.plan.max_seg <= kBlockWaves &&
                          ((int64_t)a.plan.n_seg << ls) <= (narrow_slice ? 20480 : 65536);
  const int waves = block_rows ? kBlockWaves : 4, wave_units = by_two ? kLongPerWave : 1;
  const int nvec = (a.head.d_slice + VEC - 1) / VEC;
  // One wavefront per static segment.  The kept boundary rows are a few entries each.  Where all wavefronts go on to them
  // after their segment, the launch ends in a long stretch of short rows, bound by the rate at which workgroups start, while
  // the wavefronts wait for the store of their first row (19 800 rows in four slices beside 52 800 segments: 110 of 640 us).
  // Dealt among the workgroups of the segments they go by beside the long rows (all transposed aggregates of a step, us: that graph
  // 2000 -> 1770; 25000 rows of 75 entries 255 -> 224; 90000 rows of 50 325 -> 284; 578125 rows of 22 1712 -> 1671).  But a wavefront
  // that takes a row and ends costs more than one that goes on to the next, the more so the narrower the row, and in a launch of few
  // rounds of wavefronts the long rows should start first.  The lines, as the time with two rows dealt to a wavefront over that without:
  // 13 entries a row (90000 rows of 8 414 us, dealt 430; 300000 of 11.5, 128 floats 446, 456; 60000 of 13.2 121, 101), for up to 64 floats
  // 24 (150000 of 17 176 us, dealt 185; 400000 of 16 327, 334; 60000 of 25.5 64, 60); 16384 wavefronts (12000 of 110 entries, 100 floats
  // 57 us, dealt 60); up to 32 floats 24576 and no more short rows than segments (16 floats, 20000 of 57 beside 20000 0.97 to
  // 1.03, 50000 of 238 beside 20000 0.94 to 0.99, beside 300000 1.05 to 1.11).  Two rows to a wavefront, four where there are twice as many as segments or more (one, two
  // and four: 128 floats, 50000 of 140 beside 300000 1.12, 1.05, 1.02; 48 floats, 50000 of 238 beside as many 1.09, 1.04, 1.01; 256 floats,
  // 12000 of 101 beside 1200 1.07, 1.00, 1.00; 197 758 rows beside 52 800 segments in four slices 2591, -, 2427 us).  Of 4691
  // launches of 12000 to 570000 rows this rule deals 3032, which take 0.971 of the time without, 24 of them 5 to 11 % longer; with one row to a
  // wavefront below 100000 segments and 16384 wavefronts for all widths it was 3220, 0.977 and 92.  They are dealt in groups of a workgroup
  // per XCD and slice, so that no XCD has more of them, at a share that is no simple fraction (one in six exactly: the same
  // shader engines had all of them, 1369 and 1565 us), and over every 32 groups in the order of the reversed bits, because near such a fraction
  // the same ones have all of them for hundreds of groups on end (150000 rows beside as many, 64 floats 215 -> 198, 256 floats 625 -> 565).
  const int64_t per = 8 >> ls;
  auto groups = [&](int64_t n) { return (n + per - 1) / per; };
  // Else the last wavefront of a row adds it up (finish_long_row), and waits for its store and its count first, some 2 us: where most wavefronts have such
  // a segment that costs more than the launch.  The launch and its sums / so, us: 40500 segments in four slices 434 / 440 (transposed, 31900 485 / 493), in
  // one 126 / 123 (207 / 206), 23400 in one 216 / 205, transposed 20100 in two 697 / 690, 16900 in one 791 / 785, 200 in one 28 / 23 (20011 rows).  Nothing is timed
  // between 40500 segments and slices and 127600, so the line lies where the known gains end (the 40500 are 40300 to 41500 in graphs of the same kind).  Nor
  // with rows of more segments than the 54 of these graphs: what such a row's last wavefront takes, a wait for every eight of them, has to go by beside the rows
  // of one segment, which come behind the long rows.  So no longer rows than 64 segments, unless there is a round of the chip's wavefronts for every wait.
  const bool aside = a.plan.max_seg <= kByLastMaxSegments || ((n_units - a.plan.n_part) << ls) >= (int64_t)a.plan.max_seg * (kResidentWaves / 8);
  const bool by_last = !multi_only && !block_rows && ((int64_t)a.plan.n_part << ls) <= kByLastMaxParts && aside;
  if (!by_last) a.plan.arrived = nullptr;
  if (block_rows) {  // the rows of one segment are left
    a.units += a.plan.n_part;
    a.head.n_units -= a.plan.n_part;
  }
  const int64_t unit_groups = groups((a.head.n_units + waves * wave_units - 1) / (waves * wave_units));
  const bool dealt = extra_rows >= 0 && avg_len >= (a.d > 64 ? 13 : 24) && (n_units << ls) >= (a.d > 32 ? 16384 : 24576) &&
                     (a.d > 32 || extra_rows <= n_units);
  // Eight at a time (short_rows) where they are not dealt, every wavefront has so many to go on to, and they are no fewer than the
  // segments, whose gather has two or three registers less then with 16 lanes to a row (8 and 12 bytes of scratch).  Us, one at a time -> eight: 578125 rows beside 3.1 M boundary
  // rows of 1.4 entries, 128 floats 1758 -> 1287, 66 floats 1496 -> 962, 16 floats 1392 -> 643, beside 1.54 M 1169 -> 1045, beside 308000 787 -> 787;
  // 89625 beside 211000, 512 floats 610 -> 517, 130 floats 198 -> 180; 306250 beside 746000, 48 floats 546 -> 499; beside fewer than segments 578125 beside
  // 154000, 64 floats 466 -> 503.  Dealt and by eight, 306250 beside 746000, 128 floats 964 -> 984, 29125 beside 197758, 256 floats 690 -> 667: left.
  const bool by_eight = VEC == 4 && !dealt && !block_rows && nvec <= kWave && extra_rows >= std::max<int64_t>(65536, n_units);
  int64_t extra_groups = 0;
  if (dealt) {
    const int rows = waves * (extra_rows >= 2 * n_units ? 4 : 2);
    extra_groups = groups((extra_rows + rows - 1) / rows);
    extra_groups += extra_groups / 32 + 1;  // (never none: any number is walked)
  } else if (extra_rows >= 0) {  // (as many wavefronts by eight: there are more such units than are in flight)
    extra_groups = groups(std::min<int64_t>((extra_rows + waves - 1) / waves, 8192));
  }
  const int64_t all_groups = unit_groups + extra_groups;
  a.head.n_block_rows = block_rows ? (int32_t)(groups(a.plan.n_multi) * per) : 0;
  a.head.extra_share = dealt ? (uint32_t)((((uint64_t)extra_groups << 32) + all_groups - 1) / all_groups) : 0;
  a.head.n_groups = (int32_t)all_groups;
  a.head.extra_step = (int32_t)((dealt ? extra_groups : all_groups) * per * waves);
  const unsigned each = (unsigned)(a.head.n_block_rows + all_groups * per);  // workgroups of a slice
  const size_t block_lds = (size_t)kBlockWaves * a.head.d_slice * sizeof(float);  // at most 64 KB
  const unsigned cblocks = multi_only || block_rows || by_last ? 0u : (unsigned)((a.plan.n_multi + 3) / 4);
  const int full_nvec = (a.d + VEC - 1) / VEC;
  if (each == 0) return hipSuccess;
  const unsigned blocks = each << ls;
  if (ls > 0) {
    // The slices in turn pay where a turn is long beside filling the L2 anew and the launch is several rounds of
    // workgroups (whole launches, fixed and in turn, us): 6000 rows of 250 entries and 512 floats 221 -> 215, 256 floats
    // 140 -> 138; 25000 rows of 75 entries 405 -> 397, 248 -> 240; 12000 rows of 75 192 -> 193, 121 -> 123; 50000 rows of 19
    // 367 -> 370, 226 -> 223; 6000 rows of 75 104 -> 108.
    const bool in_turn = (int64_t)avg_len * a.n_split >= 1250000 && each > (1u << ls);  // (there may be a handful of long rows alone)
    a.head.turn_share = in_turn ? (uint32_t)(((uint64_t)1 << (32 + ls)) / each) : 0;
  }
  if (a.d_store != a.d) {  // padded sources, dense narrower outputs: d < 128, four floats per lane
    if constexpr (VEC == 4 && !RAGGED) {
#define BNS_SPMM_NARROW(LPR)                                                                                \
  do {                                                                                                      \
    if (block_rows) spmm_kernel<4, 1, LPR, true, true><<<blocks, kBlockWaves * kWave, block_lds, s>>>(a); \
    else if (by_eight) spmm_kernel<4, 1, LPR, true, false, false, true><<<blocks, 256, 0, s>>>(a);        \
    else spmm_kernel<4, 1, LPR, true><<<blocks, 256, 0, s>>>(a);                                          \
  } while (0)
      if (nvec <= 4) BNS_SPMM_NARROW(4);
      else if (nvec <= 8) BNS_SPMM_NARROW(8);
      else if (nvec <= 16) BNS_SPMM_NARROW(16);
      else BNS_SPMM_NARROW(32);
#undef BNS_SPMM_NARROW
      if (cblocks) spmm_combine_kernel<4, 1, true><<<cblocks, 256, 0, s>>>(a);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
#define BNS_SPMM(MAXCH, LPR)                                                                                              \
  do {                                                                                                                    \
    if (block_rows) spmm_kernel<VEC, MAXCH, LPR, false, true, RAGGED><<<blocks, kBlockWaves * kWave, block_lds, s>>>(a); \
    else if (VEC == 4 && MAXCH == 1 && by_eight) spmm_kernel<VEC, MAXCH, LPR, false, false, RAGGED, VEC == 4 && MAXCH == 1><<<blocks, 256, 0, s>>>(a); \
    else spmm_kernel<VEC, MAXCH, LPR, false, false, RAGGED><<<blocks, 256, 0, s>>>(a);                                  \
  } while (0)
#define BNS_COMBINE(MAXCH) spmm_combine_kernel<VEC, MAXCH, false, RAGGED><<<cblocks, 256, 0, s>>>(a)
  if constexpr (VEC < 4) {
    if (nvec <= 1) BNS_SPMM(1, 1);
    else if (nvec <= 2) BNS_SPMM(1, 2);
    else if (nvec <= 4) BNS_SPMM(1, 4);
    else if (nvec <= 8) BNS_SPMM(1, 8);
    else return hipErrorInvalidValue;
    if (cblocks) BNS_COMBINE(1);
  } else {
    if (by_two) spmm_long_kernel<<<blocks, 256, 0, s>>>(a);
    else if (nvec <= 1) BNS_SPMM(1, 1);
    else if (nvec <= 2) BNS_SPMM(1, 2);
    else if (nvec <= 4) BNS_SPMM(1, 4);
    else if (nvec <= 8) BNS_SPMM(1, 8);
    else if (nvec <= 16) BNS_SPMM(1, 16);
    else if (nvec <= 32) BNS_SPMM(1, 32);
    else if (nvec <= 64) BNS_SPMM(1, 64);
    else if (nvec <= 128) BNS_SPMM(2, 64);
    else if (nvec <= 192) BNS_SPMM(3, 64);
    else if (nvec <= 256) BNS_SPMM(4, 64);
    else if (nvec <= 384) BNS_SPMM(6, 64);
    else if (nvec <= 512) BNS_SPMM(8, 64);
    else return hipErrorInvalidValue;
    if (cblocks) {
      if (full_nvec <= 64) BNS_COMBINE(1);
      else if (full_nvec <= 128) BNS_COMBINE(2);
      else if (full_nvec <= 256) BNS_COMBINE(4);
      else if (full_nvec <= 384) BNS_COMBINE(6);
      else BNS_COMBINE(8);
    }
  }
#undef BNS_COMBINE
#undef BNS_SPMM
  return hipGetLastError();
}

static hipError_t launch_spmm(const SpmmArgs &a, int64_t extra_rows, bool multi_only, int32_t avg_len, bool transposed, hipStream_t s) {
  if (a.d_store != a.d && (a.d_store < 1 || a.d_store > a.d || a.d >= 128 || a.d % 4 != 0 || a.mask_src || a.init))
    return hipErrorInvalidValue;  // padded sources: narrow rows without mask or initial value only
  if (a.d % 4 == 0) return launch_spmm_vec<4, false>(a, extra_rows, multi_only, avg_len, transposed, s);
  // Widths that are no multiple of 4: 16-byte loads at 4-byte alignment, and slices as for the others, where loads of 8 or 4 bytes
  // took up to four times as many instructions (130 floats: 65 lanes, a second load for the last one) and could not be
  // sliced.  Forward and transposed, us: 60000 rows of 45 entries, 31 floats 75 -> 62 and 130 -> 91, 66 120 -> 108 and 225 -> 144, 130
  // 232 -> 197 and 443 -> 235, 258 413 -> 403 and 660 -> 404, 602 907 -> 855 and 1235 -> 846; 20011 rows of 14, 9 floats the same,
  // 66 34 -> 28 and 45 -> 35, 130 56 -> 39 and 81 -> 50, 602 145 -> 111 and 189 -> 126.  Up to 8 floats a row is one or two
  // pieces, of which a wavefront has more than there are entries (20011 rows, 6 floats: 17.7 and 19.8 us, in pieces of 16 bytes 18.5 and 20.6).
  if (a.d > 8) return launch_spmm_vec<4, true>(a, extra_rows, multi_only, avg_len, transposed, s);
  if (a.d % 2 == 0) return launch_spmm_vec<2, false>(a, extra_rows, multi_only, avg_len, transposed, s);
  return launch_spmm_vec<1, false>(a, extra_rows, multi_only, avg_len, transposed, s);
}

hipError_t spmm_fwd(const SegPlan &plan, int32_t n_in, int32_t d, const int32_t *row_ptr,
                    const int32_t *col_idx, const float *w_in, const int32_t *w_ptr, const float *row_scale,
                    const float *H_in, const float *Hu, float *partials, float *A,
                    const SpmmRowPart &part, bool long_rows_only, bool relu, hipStream_t s, int32_t d_store) {
  SpmmArgs a = spmm_fwd_args(plan, n_in, d, row_ptr, col_idx, w_in, w_ptr, row_scale, H_in, Hu, partials, A, part);
  a.relu = relu;
  if (d_store > 0) a.d_store = d_store;
  return launch_spmm(a, -1, long_rows_only, plan.avg_len, false, s);
}

hipError_t spmm_bwd(const SegPlan &plan, int32_t n_in, int32_t n_halo, int32_t d,
                    const int32_t *t_row_ptr, const int32_t *t_col_idx, const int32_t *kept_ids,
                    const int32_t *n_kept, const float *w_in, const float *w_halo, const int32_t *halo_ptr, const float *row_scale,
                    const float *dis_halo, float s_halo, const float *dA, const float *mask_src,
                    const float *init, bool skip_self, int32_t avg_len, float *partials, float *dH_in, float *dhalo,
                    int32_t expected_halo, hipStream_t s, int32_t d_store) {
  SpmmArgs a{};
  const bool halo_rows = dhalo && n_halo > 0;
  a.plan = plan; a.n_extra_dev = halo_rows ? n_kept : nullptr; a.d = d; a.d_store = d_store > 0 ? d_store : d;
  a.row_ptr = t_row_ptr; a.col_idx = t_col_idx; a.n_split = n_in;
  a.src0 = dA; a.src1 = nullptr; a.w_in = w_in; a.w_ptr = t_row_ptr; a.w_halo = w_halo; a.halo_ptr = halo_ptr; a.partials = partials;
  a.out0 = dH_in; a.out1 = dhalo; a.out_scale0 = row_scale; a.mask_src = mask_src;
  a.kept_ids = kept_ids; a.dis_halo = dis_halo; a.s_halo = s_halo;
  a.init = init; a.skip_self = skip_self;
  return launch_spmm(a, halo_rows ? expected_halo : -1, false, avg_len, true, s);
}

// ------------------------------------------------------------------------------------------
// Static segmentation of a CSR pattern (set-up).
__global__ void __launch_bounds__(256)
seg_count_kernel(int32_t n_rows, const int32_t *__restrict__ row_ptr, int32_t *__restrict__ nseg) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= n_rows) return;
  const int len = row_ptr[v + 1] - row_ptr[v];
  nseg[v] = len <= kSegLen ? 1 : (len + kSegLen - 1) / kSegLen;
}

// which: 0 -> number of partial slots of the row (0 for single-segment rows), 1 -> multi flag
__global__ void __launch_bounds__(256)
seg_multi_kernel(int32_t n_rows, const int32_t *__restrict__ seg_ptr, int which, int32_t *__restrict__ out) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= n_rows) return;
  const int n = seg_ptr[v + 1] - seg_ptr[v];
  out[v] = n > 1 ? (which == 0 ? n : 1) : 0;
}

__global__ void __launch_bounds__(256)
seg_fill_kernel(int32_t n_rows, const int32_t *__restrict__ seg_ptr, const int32_t *__restrict__ mpos,
                const int32_t *__restrict__ part_ptr, int2 *__restrict__ seg_unit,
                int32_t *__restrict__ mrow, int2 *__restrict__ part_unit, int2 *__restrict__ order) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= n_rows) return;
  const int s0 = seg_ptr[v], s1 = seg_ptr[v + 1];
  for (int s = s0; s < s1; ++s) seg_unit[s] = make_int2(v, s1 - s0 > 1 ? part_ptr[v] + s - s0 : -1);
  if (s1 - s0 > 1) {
    mrow[mpos[v]] = v;
    for (int s = 0; s < s1 - s0; ++s) part_unit[part_ptr[v] + s] = order[part_ptr[v] + s] = make_int2(v, part_ptr[v] + s);
  } else {
    order[part_ptr[n_rows] + v - mpos[v]] = make_int2(v, -1);
  }
}

// The segments of the long rows by the column of their middle entry, in kBuckets steps: a counting sort, stable.  What bounds the
// gathers is the rate at which the L2s pull missed lines.  A segment of a row of many covers a small part of the columns, so that
// the segments in flight together share their feature rows while these are in the L2s; in the order of the rows each part of the columns
// came by again with every row.  The sums and their order are what they are in any order of the units.  Us, by row -> by column:
// 29125 rows of 340 entries, 256 floats in slices of 64 500 -> 422, beside 197758 boundary nodes all kept 842 -> 650, transposed
// 500 -> 434 and 677 -> 640; transposed 306250 rows of 45, 128 floats 763 -> 695, 578125 of 21 815 -> 789; the long rows alone, while they
// went in slices of 32, 251 -> 172 and 252 -> 184 (the slices they go in now: spmm_long_kernel).  By the column of the first entry 1 to 12 % slower (204 -> 230 for the long rows of the 306250, 100
// floats).  With an eighth of the columns to each XCD, so that a line is in one L2 alone, the long rows are no faster (175 and 193) and the
// XCDs that have the boundary columns end last (650 -> 725).  Shorter segments are narrower, but their partial sums eat that up (transposed,
// 128 entries 434 + 12 -> 418 + 22 and 789 + 9 -> 762 + 17, 64 entries 460 + 41).
// A tile is kOrderTile segments; counts[bucket * tiles + tile].
constexpr int kBuckets = 1024, kOrderTile = 4096, kOrderMin = 4096;
// Calls f(i) for the thread's own keys among the m of the tile, in ascending order, eight to a read of the LDS.  f leaves no store to memory in
// the loop: those held it up (set-up of 578125 rows 8.2 -> 7.9 ms, 7.5 without the order).
template <typename F>
__device__ __forceinline__ void each_match(const uint16_t *keys, int m, F f) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  for (int i = 0; i < m; i += 8) {
    const u4 w = *reinterpret_cast<const u4 *>(keys + i);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (((w[k / 2] >> (16 * (k & 1))) & 0xffffu) == threadIdx.x && i + k < m) f(i + k);
  }
}

__device__ __forceinline__ void segment_buckets(uint16_t *keys, int n, const int2 *units, const int32_t *row_ptr, const int32_t *col, int64_t n_cols,
                                                const int32_t *seg_ptr, const int32_t *part_ptr) {
  for (int i = threadIdx.x; i < n; i += kBuckets) {
    const int2 u = units[i];
    const int r0 = row_ptr[u.x], r1 = row_ptr[u.x + 1], nseg = seg_ptr[u.x + 1] - seg_ptr[u.x];
    const int chunk = (r1 - r0 + nseg - 1) / nseg;
    const int e = min(r0 + (u.y - part_ptr[u.x]) * chunk + chunk / 2, r1 - 1);
    keys[i] = (uint16_t)max((int64_t)0, min((int64_t)col[e] * kBuckets / n_cols, (int64_t)kBuckets - 1));
  }
  __syncthreads();
}

__global__ void __launch_bounds__(kBuckets)
seg_order_count_kernel(int n, const int2 *units, const int32_t *row_ptr, const int32_t *col, int64_t n_cols, const int32_t *seg_ptr,
                       const int32_t *part_ptr, int32_t *counts) {
  __shared__ __attribute__((aligned(16))) uint16_t keys[kOrderTile];
  const int i0 = blockIdx.x * kOrderTile, m = min(kOrderTile, n - i0);
  segment_buckets(keys, m, units + i0, row_ptr, col, n_cols, seg_ptr, part_ptr);
  int mine = 0;
  each_match(keys, m, [&](int) { ++mine; });
  counts[threadIdx.x * gridDim.x + blockIdx.x] = mine;
}

__global__ void __launch_bounds__(kBuckets)
seg_order_write_kernel(int n, const int2 *units, const int32_t *row_ptr, const int32_t *col, int64_t n_cols, const int32_t *seg_ptr,
                       const int32_t *part_ptr, const int32_t *starts, int2 *order) {
  __shared__ __attribute__((aligned(16))) uint16_t keys[kOrderTile];
  __shared__ int32_t place[kOrderTile];
  const int i0 = blockIdx.x * kOrderTile, m = min(kOrderTile, n - i0);
  segment_buckets(keys, m, units + i0, row_ptr, col, n_cols, seg_ptr, part_ptr);
  int at = starts[threadIdx.x * gridDim.x + blockIdx.x];
  each_match(keys, m, [&](int i) { place[i] = at++; });
  __syncthreads();
  for (int i = threadIdx.x; i < m; i += kBuckets) order[place[i]] = units[i0 + i];
}

// *out = the most segments of a row, over the *n multi-segment rows (1 if there is none)
__global__ void __launch_bounds__(1024)
seg_max_kernel(const int32_t *__restrict__ n, const int32_t *__restrict__ mrow, const int32_t *__restrict__ seg_ptr,
               int32_t *__restrict__ out) {
  __shared__ int part[1024 / kWave];
  int m = 1;
  for (int j = threadIdx.x; j < *n; j += 1024) m = max(m, seg_ptr[mrow[j] + 1] - seg_ptr[mrow[j]]);
  for (int off = kWave / 2; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off, kWave));
  if (lane_id() == 0) part[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 1024 / kWave; ++w) m = max(m, part[w]);
    *out = m;
  }
}

hipError_t build_seg_plan(int32_t n_rows, int64_t nnz, const int32_t *row_ptr, const int32_t *col, int64_t n_cols, SegPlan *plan,
                          int32_t *tmp_a, int32_t *tmp_b, int32_t *counts, int32_t *tile_sums, hipStream_t s) {
  const unsigned blocks = (unsigned)((n_rows + 255) / 256);
  seg_count_kernel<<<blocks, 256, 0, s>>>(n_rows, row_ptr, tmp_a);
  hipError_t e = scan_exclusive_i32(tmp_a, plan->seg_ptr, n_rows, nullptr, tile_sums, nullptr, 0, s);
  if (e != hipSuccess) return e;
  seg_multi_kernel<<<blocks, 256, 0, s>>>(n_rows, plan->seg_ptr, 0, tmp_a);
  e = scan_exclusive_i32(tmp_a, plan->part_ptr, n_rows, nullptr, tile_sums, nullptr, 0, s);
  if (e != hipSuccess) return e;
  seg_multi_kernel<<<blocks, 256, 0, s>>>(n_rows, plan->seg_ptr, 1, tmp_a);
  e = scan_exclusive_i32(tmp_a, tmp_b, n_rows, nullptr, tile_sums, nullptr, 0, s);
  if (e != hipSuccess) return e;
  seg_fill_kernel<<<blocks, 256, 0, s>>>(n_rows, plan->seg_ptr, tmp_b, plan->part_ptr, plan->seg_unit, plan->mrow,
                                         plan->part_unit, plan->order);
  seg_max_kernel<<<1, 1024, 0, s>>>(tmp_b + n_rows, plan->mrow, plan->seg_ptr, tmp_a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the totals size the launches: bring them to the host (set-up only)
  int32_t tot[4];
  e = hipMemcpyAsync(&tot[0], plan->seg_ptr + n_rows, 4, hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipMemcpyAsync(&tot[1], plan->part_ptr + n_rows, 4, hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipMemcpyAsync(&tot[2], tmp_b + n_rows, 4, hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipMemcpyAsync(&tot[3], tmp_a, 4, hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  plan->n_seg = tot[0];
  plan->n_part = tot[1];
  plan->n_multi = tot[2];
  plan->max_seg = tot[3];
  plan->avg_len = n_rows > 0 ? (int32_t)(nnz / n_rows) : 0;
  if (plan->n_part < kOrderMin) return hipSuccess;  // (all of them are in flight at once)
  const int tiles = (plan->n_part + kOrderTile - 1) / kOrderTile, n_counts = tiles * kBuckets;  // 2 n_counts <= n_part
  int32_t *const starts = counts + n_counts;                                                    // n_counts + 1
  seg_order_count_kernel<<<tiles, kBuckets, 0, s>>>(plan->n_part, plan->part_unit, row_ptr, col, n_cols, plan->seg_ptr, plan->part_ptr, counts);
  e = scan_exclusive_i32(counts, starts, n_counts, nullptr, tile_sums, nullptr, 0, s);
  if (e != hipSuccess) return e;
  seg_order_write_kernel<<<tiles, kBuckets, 0, s>>>(plan->n_part, plan->part_unit, row_ptr, col, n_cols, plan->seg_ptr, plan->part_ptr, starts,
                                                    plan->order);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Copy of a dense [n_rows, d] matrix with the rows padded by zeros to ld floats (ld a multiple of
// 4), so that an aggregate over a narrow odd width can gather with 16-byte loads.
__global__ void __launch_bounds__(256)
pad_rows_kernel(int64_t total, int32_t d, int32_t ld, const float *__restrict__ src, float *__restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int64_t r = i / ld;
  const int c = (int)(i - r * ld);
  dst[i] = c < d ? src[r * d + c] : 0.f;
}

hipError_t pad_rows(int32_t n_rows, int32_t d, int32_t ld, const float *src, float *dst, hipStream_t s) {
  if (ld < d || d < 1) return hipErrorInvalidValue;
  const int64_t total = (int64_t)n_rows * ld;
  if (total == 0) return hipSuccess;
  pad_rows_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(total, d, ld, src, dst);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Stand-in for "receive H_U" (Algorithm 1, feature exchange): the kept rows of the preloaded boundary
// features are read where they are; a record per kept node says where, and with which weight
// (S_uu = 1/p, times d~_u^-1/2 for the GCN layer).
__global__ void __launch_bounds__(256)
halo_records_kernel(const int32_t *__restrict__ kept_ids, const int32_t *__restrict__ n_kept,
                    const float *__restrict__ dis_halo, float s_halo, int2 *__restrict__ rec, int blocks,
                    const PackJobs pack) {
  if ((int)blockIdx.x >= blocks) {
    pack_unit(pack, (blockIdx.x - blocks) * 4 + (threadIdx.x >> 6));
    return;
  }
  const int n = *n_kept;
  for (int r = blockIdx.x * 256 + threadIdx.x; r < n; r += blocks * 256) {
    const int b = kept_ids[r];
    rec[r] = make_int2(b, __float_as_int(dis_halo ? s_halo * dis_halo[b] : s_halo));
  }
}

hipError_t halo_records(const int32_t *kept_ids, const int32_t *n_kept, int32_t n_halo, const float *dis_halo,
                        float s_halo, int2 *rec, const PackJobs &pack, hipStream_t s) {
  const int blocks = n_halo > 0 ? (int)std::min<int64_t>(((int64_t)n_halo + 255) / 256, 2048) : 0;
  const unsigned grid = (unsigned)(blocks + (pack.units + 3) / 4);
  if (grid == 0) return hipSuccess;
  halo_records_kernel<<<grid, 256, 0, s>>>(kept_ids, n_kept, dis_halo, s_halo, rec, blocks, pack);
  return hipGetLastError();
}

}  // namespace bns
