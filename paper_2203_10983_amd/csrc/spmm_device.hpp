// Device code shared by the aggregate kernels (Eq. 1 in the sampled matrix form of Appendix A):
// argument block, the gather of one row segment, and the scale / mask / store of a finished row.
#pragma once
#include <type_traits>

#include "device_utils.hpp"
#include "kernels.hpp"

namespace bns {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
template <int VEC, bool RAGGED = false> struct Vec;
template <> struct Vec<1> { using T = float; };
template <> struct Vec<2> { using T = v2f; };
template <> struct Vec<4> { using T = v4f; };
// RAGGED: rows of a width that is no multiple of 4 still go four floats to a lane, at any alignment of 4 bytes: the last piece
// of a row or slice is moved back to end with it, and the columns that it shares with the piece before it come out of both lanes alike.
template <> struct Vec<4, true> { using T = v4fu; };

// First column of piece iv of a row (or slice of one) of `width` floats.
template <int VEC, bool RAGGED>
__device__ __forceinline__ int piece_at(int iv, int width) {
  return RAGGED ? min(iv * VEC, width - VEC) : iv * VEC;
}
// That piece of the row at `row`.  Whole rows are indexed by pieces: with an offset in floats a gather of 33 to 64 floats took a register
// more than it has and waited for its sixth load before it asked for the last two (transposed aggregates of 46925 rows of
// 15 entries beside 93850 boundary nodes, 48 floats 75.6 -> 71.6 us, 74011 of 29 beside 148022 114.9 -> 112.6).
template <int VEC, bool RAGGED, typename F>
__device__ __forceinline__ auto *piece_of(F *row, int iv, int width) {
  using V = std::conditional_t<std::is_const_v<F>, const typename Vec<VEC, RAGGED>::T, typename Vec<VEC, RAGGED>::T>;
  if constexpr (RAGGED) return reinterpret_cast<V *>(row + piece_at<VEC, true>(iv, width));
  else return reinterpret_cast<V *>(row) + iv;
}

template <int VEC>
__device__ __forceinline__ void vec_fma(float (&acc)[VEC], float w, const float *p) {
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = fmaf(w, p[i], acc[i]);
}

struct SpmmArgs {
  SegPlan plan;                // static segmentation of rows 0..n_split-1
  // feature slicing over the XCDs (log2_slices = 0: off).  Workgroups are handed to the 8 XCDs in
  // turn, so workgroup b runs on XCD b % 8; with S = 2^log2_slices that XCD only ever touches the
  // d_slice = d / S floats of one slice of every feature row at a time, and its private L2 holds S
  // times as many distinct rows.  The slices are not equally fast:
  // where rows are a multiple of 1 KB apart, one 128-byte line in eight is gathered as if half of the L2's channels held it
  // (5.1 M random pieces of 128 bytes out of rows of 1 KB: 8000 rows 30 us, that line 37; 29125 rows 32 us, 46), and with one
  // slice for the whole launch the XCDs of that slice end last (10 M entries of 256 floats: 628 us, the others 490 to 517).
  // So an XCD takes the slices in turn.
  struct Head {                // what a workgroup needs to find its work, in one scalar load
    int32_t log2_slices, d_slice;
    uint32_t turn_share;       // turn of workgroup b of a slice: b * turn_share / 2^32 (0: the XCDs stay)
    int32_t n_units;           // work units of the kernel: segments of the plan, (row, partial-sum slot or -1)
    int32_t n_block_rows;      // BLOCK kernels: workgroups in front, of which the first n_multi own a multi-segment row of the plan each
    uint32_t extra_share;      // the *n_extra_dev further rows: share of the workgroups that are theirs alone, in 2^32 (0: none are)
    int32_t extra_step;        // wavefronts that share these rows
    int32_t n_groups;          // all groups, theirs and the units'
  } head;
  const int32_t *n_extra_dev;  // nullable: *n_extra_dev further single-segment rows follow (kept boundary)
  const int2 *units;
  int32_t d;                   // floats per gathered row = row stride of src0, src1 and the partial sums
  const int32_t *row_ptr, *col_idx;
  int32_t n_split;             // columns < n_split read src0; others src1 (weight 1)
  const float *src0, *src1;
  // Weights of the entries with a column < n_split, in the order of the static lists (null: 1).  They come first in a
  // row; the list of row v < n_split is w_ptr[v] .. w_ptr[v + 1], that of a kept boundary row at
  // w_halo + halo_ptr[its node].
  // A weight per entry, read in step with the column indices, instead of a gather from a table by column: the gather cost a
  // request of its own per entry, and the table (4 bytes per node, 2.3 MB on 578 125 nodes) was hot enough to keep
  // half of every L2 from the feature rows.  Same values, same sums; transposed aggregate of 16.6 M entries of 128 floats
  // 955 -> 838 us (bytes from the fabric 6.6 -> 5.6 GB), 32.9 M entries of 64 floats in L2 651 -> 551 us.
  const float *w_in, *w_halo;
  const int32_t *w_ptr, *halo_ptr;
  // nullable: src1 is the boundary-feature table as the caller holds it (one row per boundary
  // node) and stacked column n_split + r reads its row halo_rec[r].x with weight
  // as_float(halo_rec[r].y); else src1 holds the kept rows in kept order, already scaled
  const int2 *halo_rec;
  float *partials;             // one d-vector per segment of multi-segment rows
  // output rows < n_split: out0 (scale out_scale0[row], optional mask); others: out1
  float *out0, *out1;
  const float *out_scale0;
  const float *mask_src;
  const int32_t *kept_ids;     // out1 row r is scaled by s_halo * dis_halo[kept_ids[r]]
  const float *dis_halo;
  float s_halo;
  // optional restriction of rows < n_split to a part of their entries, and an initial value:
  const int32_t *row_skip;     // skip the first row_skip[row] entries (nullable)
  const int32_t *row_take;     // then use row_take[row] entries instead of the rest (nullable)
  const float *init;           // out0 row = scale * (init row + sum) (nullable)
  bool skip_self;              // entries with column == row contribute nothing (mean aggregator)
  bool relu;                   // rows < n_split: max(., 0) after the scale (update-first layers)
  // columns stored per output row = row stride of out0 / out1; less than d when the sources are
  // padded to a multiple of 4 floats (then no mask, no init, no slices; read by the NARROW kernels only)
  int32_t d_store;
};

// A kernel that walks many work units keeps every argument in scalar registers across its loop, and this block is
// larger than they are: the overflow went to lanes of vector registers and on to scratch memory.  unit_args() gives the block
// (the kernel's only parameter) where it lies in constant memory, anew for every unit, so that each argument is read where it is used.
using ArgBlock = const __attribute__((address_space(4))) SpmmArgs;
__device__ __forceinline__ ArgBlock &unit_args() {
  auto *p = (ArgBlock *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *p;
}

using HeadWords = int __attribute__((ext_vector_type(8), aligned(4)));
static_assert(sizeof(SpmmArgs::Head) == sizeof(HeadWords));
__device__ __forceinline__ SpmmArgs::Head unit_head() {
  const HeadWords w = *reinterpret_cast<const __attribute__((address_space(4))) HeadWords *>(&unit_args().head);
  return __builtin_bit_cast(SpmmArgs::Head, w);
}

// p[i] through the scalar cache, for an i that is the same on the whole wavefront and memory that the kernel does not write.
template <typename T>
__device__ __forceinline__ T scalar_load(const T *p, int i) {
  return reinterpret_cast<const __attribute__((address_space(4))) T *>(reinterpret_cast<uintptr_t>(p))[i];
}

__device__ __forceinline__ int2 scalar_load(const int2 *p, int i) {
  const long long x = scalar_load(reinterpret_cast<const long long *>(p), i);
  return make_int2((int)x, (int)(x >> 32));
}
__device__ __forceinline__ int2 scalar_load_pair(const int32_t *p, int i) {
  return make_int2(scalar_load(p, i), scalar_load(p, i + 1));
}

// Argument block of the forward aggregate (the transposed pass fills its own).
inline SpmmArgs spmm_fwd_args(const SegPlan &plan, int32_t n_in, int32_t d, const int32_t *row_ptr,
                              const int32_t *col_idx, const float *w_in, const int32_t *w_ptr, const float *row_scale,
                              const float *H_in, const float *Hu, float *partials, float *A,
                              const SpmmRowPart &part) {
  SpmmArgs a{};
  a.plan = plan; a.n_extra_dev = nullptr; a.d = d; a.d_store = d;
  a.row_ptr = row_ptr; a.col_idx = col_idx; a.n_split = n_in;
  a.src0 = H_in; a.src1 = Hu; a.w_in = w_in; a.w_ptr = w_ptr; a.w_halo = nullptr; a.halo_ptr = nullptr; a.partials = partials; a.halo_rec = part.halo_rec;
  a.out0 = A; a.out1 = nullptr; a.out_scale0 = row_scale; a.mask_src = nullptr;
  a.kept_ids = nullptr; a.dis_halo = nullptr; a.s_halo = 0.f;
  a.row_skip = part.row_skip; a.row_take = part.row_take; a.init = part.init;
  a.skip_self = part.skip_self;
  a.head.log2_slices = 0; a.head.d_slice = d; a.relu = false;
  return a;
}

// Scale, optional ReLU mask and store of one finished row slice held as acc[c][i].
// NARROW: the sources are padded (d_store < d), the output rows are dense with d_store columns.  width: of the slice, for RAGGED rows.
template <int VEC, int MAXCH, bool NARROW = false, bool RAGGED = false, typename Args>
__device__ __forceinline__ void finish_row(Args &a, int row, int sl, int nvec, int d_off,
                                           float (&acc)[MAXCH][VEC], int width = 0) {
  using V = typename Vec<VEC, RAGGED>::T;
  const int d = a.d, ds = NARROW ? (int)a.d_store : d;
  float scale;
  float *out;
  const float *mask = nullptr;
  const float *init = nullptr;
  if (row < a.n_split) {
    if (a.init) init = a.init + (size_t)row * d + d_off;
    scale = a.out_scale0 ? scalar_load(a.out_scale0, row) : 1.f;
    out = a.out0 + (size_t)row * ds + d_off;
    if (a.mask_src) mask = a.mask_src + (size_t)row * d + d_off;
  } else {
    if (a.out1 == nullptr) return;
    const int r = row - a.n_split;
    scale = a.dis_halo ? a.s_halo * scalar_load(a.dis_halo, scalar_load(a.kept_ids, r)) : a.s_halo;
    out = a.out1 + (size_t)r * ds + d_off;
  }
#pragma unroll
  for (int c = 0; c < MAXCH; ++c) {
    const int iv = c * kWave + sl;
    if (iv < nvec) {
      V o;
      float *po = reinterpret_cast<float *>(&o);
#pragma unroll
      for (int i = 0; i < VEC; ++i) po[i] = acc[c][i];
      if (init) {
        const V x0 = *piece_of<VEC, RAGGED>(init, iv, width);
        const float *p0 = reinterpret_cast<const float *>(&x0);
#pragma unroll
        for (int i = 0; i < VEC; ++i) po[i] += p0[i];
      }
#pragma unroll
      for (int i = 0; i < VEC; ++i) po[i] *= scale;
      if (a.relu) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) po[i] = fmaxf(po[i], 0.f);
      }
      if (mask) {
        const V m = __builtin_nontemporal_load(piece_of<VEC, RAGGED>(mask, iv, width));  // read once
        const float *pm = reinterpret_cast<const float *>(&m);
#pragma unroll
        for (int i = 0; i < VEC; ++i) po[i] = pm[i] > 0.f ? po[i] : 0.f;
      }
      if constexpr (!NARROW) {
        // streamed out: a non-temporal store leaves the L2 to the feature rows being gathered
        // (measured: 1.7 % of a training step on the largest workload)
        __builtin_nontemporal_store(o, piece_of<VEC, RAGGED>(out, iv, width));
      } else {  // padded sources: the output rows are dense and hold the first ds columns
#pragma unroll
        for (int i = 0; i < VEC; ++i)
          if (iv * VEC + i < ds) out[iv * VEC + i] = po[i];
      }
    }
  }
}

// Memory that other compute units write or read in the same launch: accesses at the agent's scope, past the caches of one XCD.  base: the same
// on the whole wavefront.
constexpr int kAgentScope = 16;  // sc1
template <int VEC, typename V>
__device__ __forceinline__ void shared_store(float *base, int at, const V &v) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const auto r = __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000);
  if constexpr (VEC == 4) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, at * 4, 0, kAgentScope);
  else if constexpr (VEC == 2) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, at * 4, 0, kAgentScope);
  else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, at * 4, 0, kAgentScope);
}
template <int VEC, typename V>
__device__ __forceinline__ V shared_load(const float *base, int at) {
  const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, -1, 0x00020000);
  if constexpr (VEC == 4) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, at * 4, 0, kAgentScope));
  else if constexpr (VEC == 2) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, at * 4, 0, kAgentScope));
  else return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, at * 4, 0, kAgentScope));
}

// Weights of a row's entries [.., end) with an inner column: w[e] for entry e (w null: 1).
struct InnerWeights {
  const float *w;
  int end;
};
template <typename Args>
__device__ __forceinline__ InnerWeights inner_weights(Args &a, int row, int r0, int r1) {  // r0, r1: its entries
  if (!a.w_in) return {nullptr, r0};
  if (row >= a.n_split) return {a.w_halo + (scalar_load(a.halo_ptr, scalar_load(a.kept_ids, row - a.n_split)) - r0), r1};
  const int2 ii = scalar_load_pair(a.w_ptr, row);
  return {a.w_in + (ii.x - r0), r0 + (ii.y - ii.x)};
}

// Feature-row address and weight of an entry with the stacked column index c of row `row`; inner(): its weight if c
// is an inner column.
template <typename F, typename Args>
__device__ __forceinline__ void entry_source(Args &a, int row, int c, int d_off,
                                             unsigned long long &p, float &w, F inner) {
  const int d = a.d;
  if (c < a.n_split) {
    p = (unsigned long long)(a.src0 + (size_t)c * d + d_off);
    w = inner();
    if (a.skip_self && c == row) w = 0.f;  // the stored self-loop is not a neighbour
  } else if (a.halo_rec) {
    const int2 r = a.halo_rec[c - a.n_split];
    p = (unsigned long long)(a.src1 + (size_t)r.x * d + d_off);
    w = __int_as_float(r.y);
  } else {
    p = (unsigned long long)(a.src1 + (size_t)(c - a.n_split) * d + d_off);
    w = 1.f;
  }
}

// Rows of at most 64 floats sit in L2 more often than not, and then the three cross-lane reads per load (two address
// halves and the weight, through the LDS pipe) bound the gather: that pipe was busy half of the time.  With 16 lanes
// per row the broadcast inside a lane group is one DPP move instead (a plain vector instruction): 685 -> 651 us on
// 32.9 M entries of 64 floats in L2, 228 -> 195 us for the padded 41-float rows of the same graph.  With 8 lanes it is two
// moves, and eight loads are in flight instead of four: 32 floats, 29125 rows of 340 entries 81 -> 78 us, with 19800
// boundary rows 123 -> 108; 100000 rows of 15 beside 50000 boundary rows 96 -> 86.  Rows of 32 lanes
// come from beyond L2 and are bound by the fabric, and the DPP form (over two rows of 16 lanes) was the slower one
// there: 836 -> 910 us on 12.8 M entries of 128 floats, one-kernel layer 694 -> 780.
constexpr bool dpp_gather(int maxch, int lpr) { return maxch == 1 && (lpr == 16 || lpr == 8); }

// Which entry of a batch of 64 a lane holds.  The wavefront walks EP = 64 / LPR entries per step, lane group g
// entry EP t + g in step t; for the DPP form that entry is held by lane t of the group.  The entries are fetched in their own
// order and change lanes afterwards: fetched where they are held, a load of 64 consecutive indices was 36 requests of
// the vector L1 instead of 4 (29125 rows of 340 entries, 256 floats in four slices 544 -> 530 us, transposed 520 -> 506).
template <int LPR, bool DPP>
__device__ __forceinline__ int batch_entry() {
  const int lane = lane_id();
  return DPP ? (lane % LPR) * (kWave / LPR) + lane / LPR : lane;
}

// The value of lane T of every row of 16 lanes, on all lanes of the row.
template <int T>
__device__ __forceinline__ unsigned row_bcast(unsigned x) {
  return (unsigned)__builtin_amdgcn_mov_dpp((int)x, 0x150 + T, 0xf, 0xf, true);  // row_newbcast:T
}

// The value of lane T of every eight lanes, on all of them: two moves, each into half of the banks of a row of 16.
template <int T>
__device__ __forceinline__ unsigned half_row_bcast(unsigned x) {
  const int a = __builtin_amdgcn_mov_dpp((int)x, 0x150 + T, 0xf, 0xf, true);
  return (unsigned)__builtin_amdgcn_update_dpp(a, (int)x, 0x158 + T, 0xf, 0xc, false);
}

// 4 VEC bytes at an address that was put together from its halves.  The address space has to be said: the compiler
// takes such a pointer for a generic one and makes a flat load of it, which also waits for the LDS pipe.
template <int VEC, bool RAGGED>
__device__ __forceinline__ typename Vec<VEC, RAGGED>::T load_row_piece(unsigned hi, unsigned lo, int at) {
  using V = typename Vec<VEC, RAGGED>::T;
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  return *reinterpret_cast<const __attribute__((address_space(1))) V *>(__builtin_bit_cast(unsigned long long, (u2){lo, hi}) + (unsigned)at * 4u);
}

// acc += sum over the cnt <= 64 entries of a batch, held one per lane (batch_entry; address p_l, weight w_l, zero past
// the end), of w * feature row.  The lanes span the feature dimension (VEC floats per lane, MAXCH pieces of 64
// lanes); with LPR < 64 lanes per row the wavefront walks EP = 64/LPR neighbours at once, UNR loads in flight, and
// every lane group keeps its own partial sums (fold_groups adds them).  width: of the slice, for RAGGED rows.
template <int VEC, int MAXCH, int LPR, bool DPP = false, bool RAGGED = false>
__device__ __forceinline__ void gather_batch(unsigned long long p_l, float w_l, int cnt, int nvec,
                                             float (&acc)[MAXCH][VEC], int width = 0) {
  using V = typename Vec<VEC, RAGGED>::T;
  static_assert(!DPP || (MAXCH == 1 && (LPR == 16 || LPR == 8)), "a feature row per DPP row of 16 lanes, or two");
  constexpr int EP = kWave / LPR;  // neighbours walked at once
  constexpr int UNR = MAXCH == 1 && (LPR >= 16 || DPP) ? 8 : 4;
  const int lane = lane_id();
  const int g = lane / LPR, sl = lane % LPR;
  const unsigned lo_l = (unsigned)p_l, hi_l = (unsigned)(p_l >> 32), w_u = __float_as_uint(w_l);
  // address and weight of this lane group's entry in step t (T: the same where it has to be a constant)
  auto bcast = [&](auto tc, int t, unsigned &lo, unsigned &hi, unsigned &w) {
    if constexpr (DPP) {
      constexpr int T = decltype(tc)::value;
      auto from = [](unsigned x) { return LPR == 16 ? row_bcast<T>(x) : half_row_bcast<T % 8>(x); };
      lo = from(lo_l);
      hi = from(hi_l);
      w = from(w_u);
    } else if constexpr (EP == 1) {
      lo = __builtin_amdgcn_readlane(lo_l, t);
      hi = __builtin_amdgcn_readlane(hi_l, t);
      w = __builtin_amdgcn_readlane(w_u, t);
    } else {
      lo = __shfl(lo_l, t * EP + g, kWave);
      hi = __shfl(hi_l, t * EP + g, kWave);
      w = __shfl(w_u, t * EP + g, kWave);
    }
  };
  // UNR steps from t0 (T0, where the step has to be a constant) on; TAIL: the batch ends among them
  auto steps = [&](auto tail, auto t0c, int t0) {
    constexpr bool TAIL = decltype(tail)::value;
    constexpr int T0 = decltype(t0c)::value;
    V v[UNR][MAXCH];
    unsigned w[UNR];
    auto step = [&](auto tc) {
      constexpr int t = decltype(tc)::value;
      if (TAIL && (t0 + t) * EP >= cnt) return;
      unsigned lo, hi;
      bcast(std::integral_constant<int, T0 + t>{}, t0 + t, lo, hi, w[t]);
#pragma unroll
      for (int c = 0; c < MAXCH; ++c) {
        const int iv = c * kWave + sl;
        if (TAIL || MAXCH > 1) {
          v[t][c] = V{};
          if ((EP == 1 || (t0 + t) * EP + g < cnt) && iv < nvec)
            v[t][c] = load_row_piece<VEC, RAGGED>(hi, lo, piece_at<VEC, RAGGED>(iv, width));
        } else {  // lanes past the row's pieces repeat the last one and store nothing
          v[t][c] = load_row_piece<VEC, RAGGED>(hi, lo, RAGGED ? piece_at<VEC, RAGGED>(iv, width) : min(iv, nvec - 1) * VEC);
        }
      }
    };
    step(std::integral_constant<int, 0>{}); step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 3>{});
    if constexpr (UNR == 8) {
      step(std::integral_constant<int, 4>{}); step(std::integral_constant<int, 5>{});
      step(std::integral_constant<int, 6>{}); step(std::integral_constant<int, 7>{});
    }
#pragma unroll
    for (int t = 0; t < UNR; ++t) {
      if (TAIL && (t0 + t) * EP >= cnt) break;
#pragma unroll
      for (int c = 0; c < MAXCH; ++c) vec_fma<VEC>(acc[c], __uint_as_float(w[t]), reinterpret_cast<const float *>(&v[t][c]));
    }
  };
  if constexpr (DPP) {
    auto chunk = [&](auto t0c) {
      constexpr int T0 = decltype(t0c)::value;
      if (T0 * EP >= cnt) return;
      if ((T0 + UNR) * EP <= cnt) steps(std::false_type{}, t0c, T0);
      else steps(std::true_type{}, t0c, T0);
    };
    chunk(std::integral_constant<int, 0>{});
    if constexpr (EP * UNR < kWave) chunk(std::integral_constant<int, 8>{});
  } else {
    int t0 = 0;
    for (; (t0 + UNR) * EP <= cnt; t0 += UNR) steps(std::false_type{}, std::integral_constant<int, 0>{}, t0);
    if (t0 * EP < cnt) steps(std::true_type{}, std::integral_constant<int, 0>{}, t0);
  }
}

// x plus the value of the lane whose number differs by `off`.
__device__ __forceinline__ float lane_pair_sum(float x, int off) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  const unsigned u = __float_as_uint(x);
  if (off == 8) return x + __int_as_float(__builtin_amdgcn_mov_dpp((int)u, 0x128, 0xf, 0xf, true));  // row_ror:8
  if (off == 16) {
    const u2 w = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(w[0]) + __uint_as_float(w[1]);
  }
  if (off == 32) {
    const u2 w = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(w[0]) + __uint_as_float(w[1]);
  }
  return x + __shfl_xor(x, off, kWave);
}

// Adds the partial sums of the 64/LPR lane groups; afterwards lane group 0 holds the total.
template <int VEC, int MAXCH, int LPR>
__device__ __forceinline__ void fold_groups(float (&acc)[MAXCH][VEC]) {
  if constexpr (kWave / LPR > 1) {
#pragma unroll
    for (int off = LPR; off < kWave; off <<= 1)
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[0][i] = lane_pair_sum(acc[0][i], off);
  }
}

// Sum of w * (feature row) over the entries [e0, e1) of `row`, at most a few hundred of them;
// lane group 0 (lanes < LPR) ends up with the result.  d_off / nvec: first feature column and
// number of VEC-pieces handled.
template <int VEC, int MAXCH, int LPR, bool RAGGED = false, typename Args>
__device__ __forceinline__ void gather_segment(Args &a, int row, const InnerWeights iw, int e0, int e1,
                                               int d_off, int nvec, float (&acc)[MAXCH][VEC], int width = 0) {
#pragma unroll
  for (int c = 0; c < MAXCH; ++c)
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[c][i] = 0.f;
  for (int base = e0; base < e1; base += kWave) {
    const int cnt = min(kWave, e1 - base);
    // one neighbour per lane: its feature-row address and weight
    unsigned long long p_l = 0;
    float w_l = 0.f;
    constexpr bool DPP = !RAGGED && dpp_gather(MAXCH, LPR);  // (ragged ones would spill three registers)
    const int lane = lane_id();
    int c = 0;
    float w_e = 0.f;
    if (lane < cnt) {
      const int e = base + lane;
      if (e < iw.end) w_e = iw.w[e];  // (asked for beside the column index, not after it)
      c = a.col_idx[e];
    }
    const int mine = batch_entry<LPR, DPP>();
    if (DPP) {
      c = __shfl(c, mine, kWave);
      w_e = __shfl(w_e, mine, kWave);
    }
    if (mine < cnt) entry_source(a, row, c, d_off, p_l, w_l, [&] { return iw.w ? w_e : 1.f; });
    gather_batch<VEC, MAXCH, LPR, DPP, RAGGED>(p_l, w_l, cnt, nvec, acc, width);
  }
  fold_groups<VEC, MAXCH, LPR>(acc);
}

// The kept boundary rows r0 .. r0 + n - 1, n <= kShortRows, of a transposed aggregate: a few entries each, one after another in the CSR.
// A row at a time is a chain of four reads that hang on each other (row start, node and its list, column, features) beside a few
// hundred bytes of data.  Here the lanes fetch what the rows and all their entries need at once, and the first two steps of four
// rows are in flight together.  The order of every sum is that of gather_segment.
// For rows of at most 64 entries together.
constexpr int kShortRows = 8;
template <int VEC, int LPR, bool NARROW, bool RAGGED, typename Args>
__device__ __forceinline__ void short_rows(Args &a, int r0, int n, int d_off, int nvec, int width) {
  using V = typename Vec<VEC, RAGGED>::T;
  constexpr int EP = kWave / LPR;
  int lane = lane_id();
  asm volatile("" : "+v"(lane));  // (nothing that follows from it is kept in registers beside the segments' gather)
  const int g = lane / LPR, sl = lane % LPR;
  const int d = a.d, ds = NARROW ? (int)a.d_store : d;
  const int start = a.row_ptr[a.n_split + r0 + min(lane, n)];
  const int node = a.kept_ids[r0 + min(lane, n - 1)];
  const int list = a.w_in ? a.halo_ptr[node] : 0;
  const float scale_l = a.dis_halo ? a.s_halo * a.dis_halo[node] : a.s_halo;
  auto store = [&](int i, float (&acc)[1][VEC]) {
    const float scale = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scale_l), i));
    if (g != 0 || sl >= nvec) return;
    float *const out = a.out1 + (size_t)(r0 + i) * ds + d_off;
    V o;
    float *po = reinterpret_cast<float *>(&o);
#pragma unroll
    for (int k = 0; k < VEC; ++k) po[k] = acc[0][k] * scale;
    if constexpr (!NARROW) {
      __builtin_nontemporal_store(o, piece_of<VEC, RAGGED>(out, sl, width));
    } else {
#pragma unroll
      for (int k = 0; k < VEC; ++k)
        if (sl * VEC + k < ds) out[sl * VEC + k] = po[k];
    }
  };
  const int first = __builtin_amdgcn_readlane(start, 0), total = __builtin_amdgcn_readlane(start, n) - first;  // <= 64
  // an entry per lane
  unsigned lo_l = 0, hi_l = 0, w_l = 0;
  int place = 0;  // of its weight
  for (int i = 0; i < n; ++i) {
    const int e0 = __builtin_amdgcn_readlane(start, i), l0 = __builtin_amdgcn_readlane(list, i);
    place = first + lane >= e0 ? l0 + (first + lane - e0) : place;
  }
  if (lane < total) {
    const int c = a.col_idx[first + lane];
    const float w = a.w_in ? a.w_halo[place] : 1.f;
    const unsigned long long p = (unsigned long long)(a.src0 + (size_t)c * d + d_off);
    lo_l = (unsigned)p;
    hi_l = (unsigned)(p >> 32);
    w_l = __float_as_uint(w);
  }
  auto piece = [&](int e, bool in, float &w) {  // of entry e of the batch
    const unsigned lo = __shfl(lo_l, e, kWave), hi = __shfl(hi_l, e, kWave), wu = __shfl(w_l, e, kWave);
    V v{};
    w = 0.f;
    if (in && sl < nvec) {
      v = load_row_piece<VEC, RAGGED>(hi, lo, piece_at<VEC, RAGGED>(sl, width));
      w = __uint_as_float(wu);
    }
    return v;
  };
  for (int i0 = 0; i0 < n; i0 += 4) {
    V v[4];
    float w[4];
    auto row = [&](int k, int &at, int &cnt) {
      const int i = min(i0 + k, n - 1);
      at = __builtin_amdgcn_readlane(start, i) - first;
      cnt = __builtin_amdgcn_readlane(start, i + 1) - first - at;
    };
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      int at, cnt;
      row(k, at, cnt);
      v[k] = piece(at + g, g < cnt, w[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i0 + k < n) {
        int at, cnt;
        row(k, at, cnt);
        float acc[1][VEC];
#pragma unroll
        for (int j = 0; j < VEC; ++j) acc[0][j] = 0.f;
        vec_fma<VEC>(acc[0], w[k], reinterpret_cast<const float *>(&v[k]));
        for (int t = 1; t * EP < cnt; t += 3) {
          V x[3];
          float y[3];
#pragma unroll
          for (int j = 0; j < 3; ++j) x[j] = piece(at + (t + j) * EP + g, (t + j) * EP + g < cnt, y[j]);
#pragma unroll
          for (int j = 0; j < 3; ++j) vec_fma<VEC>(acc[0], y[j], reinterpret_cast<const float *>(&x[j]));
        }
        fold_groups<VEC, 1, LPR>(acc);
        store(i0 + k, acc);
      }
    }
  }
}

}  // namespace bns
