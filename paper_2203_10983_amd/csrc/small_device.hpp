// Device code of the selection and subgraph steps of a small partition: see small.hip.
#pragma once
#include "device_utils.hpp"
#include "kernels.hpp"

namespace bns {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWords = kSmallMaxHalo / kWave;

// A barrier behind which the other threads' writes to LDS are seen (their stores to memory need not be).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// All of it, on one workgroup of kSmallThreads.  For up to NB x 1024 boundary nodes and NE x 1024 boundary entries.
template <int NB, int NE>
__device__ __forceinline__ void sample_and_build(const SmallArgs &a) {
  constexpr int kWaves = kSmallThreads / kWave;
  __shared__ uint64_t words[NB * kWaves];        // keep bits, one word per 64 boundary nodes
  __shared__ int word_prefix[kSmallWords + 1];   // kept nodes before each word; [kSmallWords] = all
  // of each kept node: its static list; the length of its list, then the entries before its transposed row
  __shared__ uint16_t kept_src[NB * kSmallThreads], kept_pos[NB * kSmallThreads + 1];
  __shared__ uint16_t kept_before[NE * kSmallThreads + 1];  // kept boundary entries before each one
  __shared__ int counts[NE * kWaves];            // kept boundary entries per wavefront and stretch of 1024
  __shared__ int wave_tot[kWaves];
  static_assert(NB * kWaves <= kSmallWords && kSmallWords == 2 * kWave && NE * kSmallThreads < 65536);
  const int t = threadIdx.x, lane = lane_id(), wid = t / kWave;
  const int n_words = (a.n_halo + kWave - 1) / kWave;
  // stretches of 1024 boundary nodes and entries: the loops over them are unrolled, and left together
  const int nb = (a.n_halo + kSmallThreads - 1) / kSmallThreads, ne = (a.e_bd + kSmallThreads - 1) / kSmallThreads;

  // ---- what the stages read of the static arrays ---------------------------------------------
  const uint32_t epoch = a.epoch_dev ? *a.epoch_dev : a.epoch;
  int64_t gid[NB];
  int list0[NB], list1[NB];
  float dis[NB];
  int bd_b[NE], bd_end[NE];  // bd_end: first the entry's row, then the end of that row's inner entries
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (i >= nb) break;
    const int b = i * kSmallThreads + t;
    if (b < a.n_halo) gid[i] = a.halo_gid[b];
  }
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    if (i >= ne) break;
    const int k = i * kSmallThreads + t;
    bd_b[i] = 0;
    if (k < a.e_bd) {
      bd_b[i] = a.sp.bd_b[k];
      bd_end[i] = a.sp.bd_row[k];
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (i >= nb) break;
    const int b = i * kSmallThreads + t;
    if (b < a.n_halo) {
      list0[i] = a.halo_ptr[b];
      list1[i] = a.halo_ptr[b + 1];
      dis[i] = a.dis_halo ? a.dis_halo[b] : 1.f;
    }
  }
  const int v0 = min(t, a.n_in), j0 = min(t, a.e_in - 1);
  const int row_inner0 = a.sp.inner_ptr[v0], row_bd0 = a.sp.bd_ptr[v0];
  const int col0 = a.sp.in_col[j0], col_bd0 = a.sp.in_bdp[j0];

  // ---- keep bits -------------------------------------------------------------------------------
  unsigned keeps = 0;  // bit i: of this thread's i-th boundary node
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (i >= nb) break;
    const int b = i * kSmallThreads + t;
    bool keep = false;
    if (b < a.n_halo) {
      uint32_t c0 = (uint32_t)gid[i], c1 = (uint32_t)((uint64_t)gid[i] >> 32), c2 = epoch, c3 = a.part_id;
      philox4x32_10(c0, c1, c2, c3, a.k0, a.k1);
      keep = (uint64_t)c0 < a.threshold;
    }
    keeps |= (unsigned)keep << i;
    const uint64_t word = __ballot(keep);
    if (lane == 0 && b < a.n_halo) {
      words[b >> 6] = word;
      a.ballots[b >> 6] = word;
    }
  }
#pragma unroll
  for (int i = 0; i < NE; ++i)
    if (i < ne && i * kSmallThreads + t < a.e_bd) bd_end[i] = a.sp.inner_ptr[bd_end[i] + 1];
  lds_barrier();
  if (wid == 0) {
    const int c0 = 2 * lane < n_words ? __popcll(words[2 * lane]) : 0, c1 = 2 * lane + 1 < n_words ? __popcll(words[2 * lane + 1]) : 0;
    const int inc = wave_inclusive_scan(c0 + c1);
    word_prefix[2 * lane] = inc - c1 - c0;
    word_prefix[2 * lane + 1] = inc - c1;
    if (lane == kWave - 1) word_prefix[kSmallWords] = inc;
  }
  lds_barrier();
  const int n_kept = word_prefix[kSmallWords];
  if (t == 0) *a.n_kept = n_kept;
  auto rank_of = [&](int b) -> int {  // rank of a kept boundary node
    return word_prefix[b >> 6] + __popcll(words[b >> 6] & ((1ull << (b & 63)) - 1ull));
  };

  // ---- kept list, remap ------------------------------------------------------------------------
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (i >= nb) break;
    const int b = i * kSmallThreads + t;
    if (b >= a.n_halo) continue;
    if ((keeps >> i) & 1u) {
      const int r = rank_of(b);
      kept_src[r] = (uint16_t)list0[i];
      kept_pos[r] = (uint16_t)(list1[i] - list0[i]);
      a.kept_ids[r] = b;
      a.rec[r] = make_int2(b, __float_as_int(a.dis_halo ? a.s_halo * dis[i] : a.s_halo));
      a.remap[b] = r;
    } else {
      a.remap[b] = -1;
    }
  }

  // ---- boundary entries: kept ones to their place ------------------------------------------------
  uint64_t kept_in_wave[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    if (i >= ne) break;
    const bool kept = i * kSmallThreads + t < a.e_bd && ((words[bd_b[i] >> 6] >> (bd_b[i] & 63)) & 1ull);
    kept_in_wave[i] = __ballot(kept);
    if (lane == 0) counts[i * kWaves + wid] = __popcll(kept_in_wave[i]);
  }
  lds_barrier();
  {
    constexpr int kPer = kWave / kWaves;  // stretches whose counts a wavefront holds at a time
    int all_kept = 0, base = 0;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      if (i >= ne) break;
      if (i % kPer == 0) {
        const int c = i * kWaves + lane < ne * kWaves ? counts[i * kWaves + lane] : 0, inc = wave_inclusive_scan(c);
        base = all_kept + inc - c;
        all_kept += __shfl(inc, kWave - 1, kWave);
      }
      const int before = __shfl(base, i % kPer * kWaves + wid, kWave);
      const int pos = before + __popcll(kept_in_wave[i] & ((1ull << lane) - 1ull));
      const int k = i * kSmallThreads + t;
      if (k < a.e_bd) {
        kept_before[k] = (uint16_t)pos;
        if ((kept_in_wave[i] >> lane) & 1ull) a.col_idx[bd_end[i] + pos] = a.n_in + rank_of(bd_b[i]);
      }
    }
    if (t == 0) kept_before[a.e_bd] = (uint16_t)all_kept;
  }

  // ---- rows of the kept nodes in the transposed subgraph: starts = prefix sum of list lengths ----
  int run = a.e_in;
  for (int r0 = 0; r0 < n_kept; r0 += kSmallThreads) {
    const int r = r0 + t, len = r < n_kept ? kept_pos[r] : 0;
    const int inc = wave_inclusive_scan(len);
    if (lane == kWave - 1) wave_tot[wid] = inc;
    lds_barrier();
    const int wave_inc = wave_inclusive_scan(lane < kWaves ? wave_tot[lane] : 0);
    const int at = run + inc - len + (wid > 0 ? __shfl(wave_inc, wid - 1, kWave) : 0);
    if (r < n_kept) {
      kept_pos[r] = (uint16_t)(at - a.e_in);
      a.kept_start[r] = at;
      a.t_tail_ptr[r] = at;
    }
    run += __shfl(wave_inc, kWaves - 1, kWave);
    lds_barrier();  // the sums are read before the next ones
  }
  if (t == 0) {
    a.kept_start[n_kept] = run;
    a.t_tail_ptr[n_kept] = run;
  }
  if (t == 0) kept_pos[n_kept] = (uint16_t)(run - a.e_in);
  lds_barrier();  // kept_before and kept_pos are read below by other threads than their writers

  // ---- row starts and inner entries --------------------------------------------------------------
  if (t <= a.n_in) a.row_ptr[t] = row_inner0 + kept_before[row_bd0];
  for (int v = kSmallThreads + t; v <= a.n_in; v += kSmallThreads) a.row_ptr[v] = a.sp.inner_ptr[v] + kept_before[a.sp.bd_ptr[v]];
  if (t == 0) *a.nnz = a.e_in + kept_before[a.e_bd];
  if (t < a.e_in) a.col_idx[t + kept_before[col_bd0]] = col0;
  for (int j0 = kSmallThreads + t; j0 < a.e_in; j0 += 4 * kSmallThreads) {  // four reads in flight
    int col[4], bd[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = min(j0 + i * kSmallThreads, a.e_in - 1);
      col[i] = a.sp.in_col[j];
      bd[i] = a.sp.in_bdp[j];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = j0 + i * kSmallThreads;
      if (j < a.e_in) a.col_idx[j + kept_before[bd[i]]] = col[i];
    }
  }

  for (int i = t; i < n_kept * 8; i += kSmallThreads) {  // eight lanes copy one list
    const int r = i >> 3, sub = i & 7;
    const int src = kept_src[r], dst = kept_pos[r], len = kept_pos[r + 1] - dst;
    for (int k = sub; k < len; k += 8) a.t_col_idx[a.e_in + dst + k] = a.halo_col[src + k];
  }
}

}  // namespace bns
