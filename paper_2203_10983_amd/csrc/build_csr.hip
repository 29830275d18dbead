// Node-induced subgraph on the inner nodes plus the kept boundary nodes (Algorithm 1, subgraph
// step), as a canonical CSR, and its transpose for the backward pass.
//
// Columns are ascending in a row, so the boundary entries are each row's tail.  Once, at set-up,
// the static CSR is split into its inner entries and its boundary entries (both row-major, each
// with its row).  Per epoch only the boundary entries are filtered (the work is proportional to
// the number of boundary edges, Appendix D): an entry-parallel prefix sum over their keep flags
// gives every kept boundary entry, every inner entry and every row start its final position
// without any per-row loop, so power-law rows cost nothing extra.
//
//   kpos[k]     = kept boundary entries before boundary entry k, from the keep flags, their counts per tile and
//                 within a tile per word
//   row_ptr[v]  = inner_ptr[v] + kpos[bd_ptr[v]]
//   inner entry j of row v      -> col_idx[j + kpos[bd_ptr[v]]]
//   kept boundary entry k, row v -> col_idx[inner_ptr[v+1] + kpos[k]]
#include <algorithm>

#include "build_device.hpp"

namespace bns {

constexpr int kThreads = 256;

// ---------------------------------------------------------------------------------- set-up
__global__ void __launch_bounds__(kThreads)
count_inner_kernel(int32_t n_in, const int32_t *__restrict__ row_ptr0,
                   const int32_t *__restrict__ col0, int32_t *__restrict__ n_inner) {
  const int v = blockIdx.x * kThreads + threadIdx.x;
  if (v >= n_in) return;
  int lo = row_ptr0[v], hi = row_ptr0[v + 1];
  const int start = lo;
  while (lo < hi) {  // first entry whose column is a boundary column
    const int mid = (lo + hi) >> 1;
    if (col0[mid] < n_in) lo = mid + 1; else hi = mid;
  }
  n_inner[v] = lo - start;
}

// One wavefront per row scatters the row's entries into the inner and boundary lists.
__global__ void __launch_bounds__(kThreads)
split_entries_kernel(int32_t n_in, const int32_t *__restrict__ row_ptr0,
                     const int32_t *__restrict__ col0, const int32_t *__restrict__ inner_ptr,
                     int32_t *__restrict__ bd_ptr, int32_t *__restrict__ in_col,
                     int32_t *__restrict__ in_bdp, int32_t *__restrict__ bd_b,
                     int32_t *__restrict__ bd_row) {
  const int lane = lane_id();
  const int waves = gridDim.x * (kThreads / kWave);
  for (int v = blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave; v <= n_in; v += waves) {
    if (v == n_in) {
      if (lane == 0) bd_ptr[n_in] = row_ptr0[n_in] - inner_ptr[n_in];
      continue;
    }
    const int e0 = row_ptr0[v], e1 = row_ptr0[v + 1];
    const int i0 = inner_ptr[v], ni = inner_ptr[v + 1] - i0;
    const int b0 = e0 - i0;
    if (lane == 0) bd_ptr[v] = b0;
    for (int e = e0 + lane; e < e1; e += kWave) {
      const int c = col0[e];
      const int o = e - e0;
      if (o < ni) { in_col[i0 + o] = c; in_bdp[i0 + o] = b0; }
      else { bd_b[b0 + o - ni] = c - n_in; bd_row[b0 + o - ni] = v; }
    }
  }
}

__global__ void __launch_bounds__(kThreads)
degree_rsqrt_kernel(const int32_t *__restrict__ deg, int32_t n, float *__restrict__ dis) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i < n) dis[i] = 1.0f / sqrtf((float)deg[i]);
}

__global__ void __launch_bounds__(kThreads)
degree_inverse_kernel(const int32_t *__restrict__ deg, int32_t n, float *__restrict__ inv) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i < n) inv[i] = deg[i] > 1 ? 1.0f / (float)(deg[i] - 1) : 0.f;
}

hipError_t degree_inverse(const int32_t *deg, int32_t n, float *inv, hipStream_t s) {
  if (n > 0) degree_inverse_kernel<<<(n + kThreads - 1) / kThreads, kThreads, 0, s>>>(deg, n, inv);
  return hipGetLastError();
}

hipError_t degree_rsqrt(const int32_t *deg, int32_t n, float *dis, hipStream_t s) {
  if (n > 0) degree_rsqrt_kernel<<<(n + kThreads - 1) / kThreads, kThreads, 0, s>>>(deg, n, dis);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kThreads)
entry_weights_kernel(int64_t n, const int32_t *__restrict__ col, const float *__restrict__ of, float *__restrict__ w) {
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (j < n) w[j] = of[col[j]];
}

hipError_t entry_weights(int64_t n, const int32_t *col, const float *of, float *w, hipStream_t s) {
  if (n > 0) entry_weights_kernel<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(n, col, of, w);
  return hipGetLastError();
}

hipError_t build_static_split(int32_t n_in, const int32_t *row_ptr0, const int32_t *col0,
                              const StaticSplit &sp, int32_t *tile_sums, hipStream_t s) {
  count_inner_kernel<<<(n_in + kThreads - 1) / kThreads, kThreads, 0, s>>>(n_in, row_ptr0, col0,
                                                                           sp.n_inner);
  hipError_t e = scan_exclusive_i32(sp.n_inner, sp.inner_ptr, n_in, nullptr, tile_sums, nullptr, 0, s);
  if (e != hipSuccess) return e;
  const int blocks = (n_in + 1 + (kThreads / kWave) - 1) / (kThreads / kWave);
  split_entries_kernel<<<blocks < 65536 ? blocks : 65536, kThreads, 0, s>>>(
      n_in, row_ptr0, col0, sp.inner_ptr, sp.bd_ptr, sp.in_col, sp.in_bdp, sp.bd_b, sp.bd_row);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------- per epoch
__global__ void __launch_bounds__(kBdThreads)
bd_count_kernel(const BdCount c, const uint64_t *__restrict__ ballots) {
  bd_count_tile(c, ballots, blockIdx.x);
}

struct StaticRows {
  const int32_t *ptr, *col;
  int32_t *t_row_ptr, *t_col_idx;
};

template <int NT>
__device__ __forceinline__ void copy_static(const StaticRows &st, int32_t n_in, int64_t e_in, int block, int n_blocks) {
  for (int64_t i = (int64_t)block * NT + threadIdx.x; i < n_in + 1 + e_in; i += (int64_t)n_blocks * NT) {
    if (i <= n_in) st.t_row_ptr[i] = st.ptr[i];
    else st.t_col_idx[i - n_in - 1] = st.col[i - n_in - 1];
  }
}

struct BuildArgs {
  // the inner entries and the row starts of the sampled CSR
  int32_t n_in;
  int64_t e_in;
  const int32_t *inner_ptr, *bd_ptr, *in_col, *in_bdp;
  int32_t *row_ptr, *nnz;
  int entry_blocks, row_blocks;
  // its kept boundary entries
  BdCount bd;
  int bd_tiles;
  const int32_t *bd_row, *remap;
  int32_t *col_idx;
  // rows of the kept boundary nodes in the transposed CSR
  const int32_t *n_kept, *kept_ids, *halo_ptr, *halo_col, *kept_start;
  int32_t *t_tail_ptr, *t_col_idx;
  int list_blocks;
  // the rows of the inner nodes in the transposed CSR, which never change (the transpose of the inner-inner block), where the
  // destination does not hold them yet
  StaticRows st;
  int copy_blocks;
};

// Places of a tile's boundary entries, from the keep flags: those inside a pass come from the population count of
// the lower lanes' bits.  The 4-byte rank is only fetched for the kept ones.
__device__ __forceinline__ void bd_fill_tile(const BuildArgs &a, int tile) {
  const int lane = lane_id(), wid = threadIdx.x / kWave;
  const int64_t base = (int64_t)tile * kScanTile + (int64_t)wid * (kBdPasses * kWave);
  unsigned long long mask[kBdPasses];
  int word_before[kBdPasses];
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i) {
    const bool in = base + i * kWave < a.bd.e_bd;
    mask[i] = in ? a.bd.mask[(base >> 6) + i] : 0ull;
    word_before[i] = in ? a.bd.before[(base >> 6) + i] : 0;
  }
  // the reads of a stage all at once: they hang on each other (node and row, rank and place)
  const unsigned long long lower = (1ull << lane) - 1ull;
  int node[kBdPasses], row[kBdPasses];
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i) {
    const int64_t k = base + i * kWave + lane;
    const bool kept = (mask[i] >> lane) & 1ull;  // (then k < e_bd)
    node[i] = kept ? a.bd.bd_b[k] : 0;
    row[i] = kept ? a.bd_row[k] : 0;
  }
  // kept boundary entries in the tiles before this one: summed here from the raw per-tile counts (ends with a barrier)
  int before[1], total[1];
  tiles_before<kBdThreads, 1>(a.bd.sums, tile, a.bd_tiles, false, before, total);
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i)
    if ((mask[i] >> lane) & 1ull) {
      node[i] = a.n_in + a.remap[node[i]];
      row[i] = a.inner_ptr[row[i] + 1];
    }
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i)
    if ((mask[i] >> lane) & 1ull) a.col_idx[row[i] + before[0] + word_before[i] + __popcll(mask[i] & lower)] = node[i];
}

// sum[i] of the thread: kept boundary entries of the tiles from `first` up to tile at(i), at most `last`, for N values of i.  Added up by the whole
// workgroup, a span of tiles at a time.  (What the thread finds stays in LDS: the ordinary case has no register to spare for it.)
constexpr int kSpanItems = 4, kSpan = kSpanItems * kBdThreads;
template <int N, typename F>
__device__ __forceinline__ void tiles_between(const BuildArgs &a, int first, int last, F at, int (*sum)[kBdThreads]) {
  __shared__ int until[kSpan];  // kept entries of the span's tiles before each one
#pragma unroll
  for (int i = 0; i < N; ++i) sum[i][threadIdx.x] = 0;
#pragma unroll 1
  for (int t0 = first; t0 < last; t0 += kSpan) {
    int x[kSpanItems], mine = 0, all;
#pragma unroll
    for (int j = 0; j < kSpanItems; ++j) {
      const int t = t0 + threadIdx.x * kSpanItems + j;
      x[j] = t < last ? a.bd.sums[t] : 0;
      mine += x[j];
    }
    int run = block_exclusive_scan<kBdThreads>(mine, &all);
#pragma unroll
    for (int j = 0; j < kSpanItems; ++j) {
      until[threadIdx.x * kSpanItems + j] = run;
      run += x[j];
    }
    __syncthreads();
#pragma unroll 1
    for (int i = 0; i < N; ++i) {
      const int t = at(i);
      sum[i][threadIdx.x] += t >= t0 + kSpan ? all : t > t0 ? until[t - t0] : 0;
    }
    __syncthreads();
  }
}

// kpos[k[i]] of a workgroup's boundary entries k[i] <= e_bd, k_first to k_last: the kept entries of the tiles before, of the words
// before in the tile, of the word's lower bits.
template <int N, bool TOGETHER>
__device__ __forceinline__ void kept_before(const BuildArgs &a, int64_t k_first, int64_t k_last, int (&k)[N]) {
  const int64_t e_bd = a.bd.e_bd;
  const int first = (int)min(k_first / kScanTile, (int64_t)a.bd_tiles - 1);
  __shared__ int between[TOGETHER ? N : 1][kBdThreads];
  if constexpr (TOGETHER)
    tiles_between<N>(a, first, (int)(min(k_last, e_bd - 1) / kScanTile), [&](int i) { return (int)(min((int64_t)k[i], e_bd - 1) / kScanTile); }, between);
  unsigned long long mask[N];
  int word[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int64_t w = min((int64_t)k[i], e_bd - 1) >> 6;
    mask[i] = a.bd.mask[w];
    word[i] = a.bd.before[w];
  }
  int before[1], total[1];
  tiles_before<kBdThreads, 1>(a.bd.sums, first, a.bd_tiles, false, before, total);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int64_t at = min((int64_t)k[i], e_bd - 1);
    int sum = before[0] + word[i];
    if constexpr (TOGETHER) sum += between[i][threadIdx.x];
    else
#pragma unroll 4
      for (int t = first; t < (int)(at / kScanTile); ++t) sum += a.bd.sums[t];
    // (bits past the last entry are clear)
    const int bit = (int)(at & 63);
    k[i] = sum + __popcll(mask[i] & ((1ull << bit) - 1ull)) + (k[i] > at ? (int)((mask[i] >> bit) & 1ull) : 0);
  }
}
// A workgroup's entries lie in a tile or a few, and a thread adds up the tiles between the first one and its own by itself.  Where boundary
// entries far outnumber rows and inner entries they lie in thousands of tiles: there the workgroup adds them up together (2000 rows of
// 4000 and of 16000 boundary entries, us: 199 -> 33 and 859 -> 142).
constexpr int kTilesAlone = 16;
template <int N>
__device__ __forceinline__ void kept_before(const BuildArgs &a, int64_t k_first, int64_t k_last, int (&k)[N]) {
  if (k_last - k_first <= kTilesAlone * kScanTile) kept_before<N, false>(a, k_first, k_last, k);
  else kept_before<N, true>(a, k_first, k_last, k);
}

// Rows of the kept boundary nodes in the transposed CSR: kept node r (boundary node b =
// kept_ids[r]) gets b's static list of inner neighbours.  Where each row starts was settled by the
// sampler (a prefix sum of the list lengths in kept order, kept_start[0..n_kept]); eight lanes copy
// one list and write the row's start.  The lists that are too long for eight lanes are left to the whole workgroup
// (197 758 boundary nodes with up to 5 800 neighbours: 81 us with eight lanes for each list, now 16).
constexpr int kLongList = 256;
constexpr int kListsPerBlock = kBdThreads / 8;
__device__ __forceinline__ void kept_rows_fill(const BuildArgs &a, int block, int n_blocks) {
  __shared__ int n_long, long_src[kListsPerBlock], long_len[kListsPerBlock], long_dst[kListsPerBlock];
  const int sub = threadIdx.x & 7;
  const int n = *a.n_kept;
  if (block == 0 && threadIdx.x == 0) a.t_tail_ptr[n] = a.kept_start[n];
  for (int r0 = block * kListsPerBlock; r0 < n; r0 += n_blocks * kListsPerBlock) {  // trip count uniform over the block
    if (threadIdx.x == 0) n_long = 0;
    __syncthreads();
    const int r = r0 + (threadIdx.x >> 3);
    if (r < n) {
      const int b = a.kept_ids[r];
      const int src = a.halo_ptr[b], len = a.halo_ptr[b + 1] - src;
      const int dst = a.kept_start[r];
      if (sub == 0) a.t_tail_ptr[r] = dst;
      if (len <= kLongList) {
        for (int i = sub; i < len; i += 8) a.t_col_idx[dst + i] = a.halo_col[src + i];
      } else if (sub == 0) {
        const int q = atomicAdd(&n_long, 1);
        long_src[q] = src;
        long_len[q] = len;
        long_dst[q] = dst;
      }
    }
    __syncthreads();
    for (int q = 0; q < n_long; ++q)
#pragma unroll 4
      for (int i = threadIdx.x; i < long_len[q]; i += kBdThreads)
        a.t_col_idx[long_dst[q] + i] = a.halo_col[long_src[q] + i];
    __syncthreads();
  }
}

constexpr int kEntryPasses = 4, kEntryTile = kEntryPasses * kBdThreads;

// Row starts and inner entries follow in closed form from the keep flags: row v's entries move down by the kept boundary entries of the
// rows before it, kpos[bd_ptr[v]], and every inner entry carries its row's bd_ptr.
__device__ __forceinline__ void inner_entries(const BuildArgs &a, int block) {
  // the reads of a stage all at once: they hang on each other (in_bdp, flags, place)
  const int64_t tile0 = (int64_t)block * kEntryTile, j0 = tile0 + threadIdx.x;
  int c[kEntryPasses], k[kEntryPasses];
#pragma unroll
  for (int i = 0; i < kEntryPasses; ++i) {
    const int64_t j = min(j0 + i * kBdThreads, a.e_in - 1);
    c[i] = a.in_col[j];
    k[i] = a.in_bdp[j];
  }
  if (a.bd.e_bd > 0) kept_before(a, a.in_bdp[tile0], a.in_bdp[min(tile0 + kEntryTile, a.e_in) - 1], k);
#pragma unroll
  for (int i = 0; i < kEntryPasses; ++i)
    if (j0 + i * kBdThreads < a.e_in) a.col_idx[j0 + i * kBdThreads + k[i]] = c[i];
}

__device__ __forceinline__ void row_starts(const BuildArgs &a, int block) {
  const int v0 = block * kEntryTile;  // (n_in + kEntryTile fits)
  int r[kEntryPasses], k[kEntryPasses];
#pragma unroll
  for (int i = 0; i < kEntryPasses; ++i) {
    const int v = min(v0 + i * kBdThreads + (int)threadIdx.x, a.n_in);
    r[i] = a.inner_ptr[v];
    k[i] = a.bd_ptr[v];
  }
  if (a.bd.e_bd > 0) kept_before(a, a.bd_ptr[v0], a.bd_ptr[min(v0 + kEntryTile - 1, a.n_in)], k);
#pragma unroll
  for (int i = 0; i < kEntryPasses; ++i) {
    const int v = v0 + i * kBdThreads + (int)threadIdx.x;
    if (v <= a.n_in) a.row_ptr[v] = r[i] + k[i];
    if (v == a.n_in) *a.nnz = r[i] + k[i];
  }
}

// Everything at once: what one part needs of another, the places of the entries, it counts again from the keep flags.  With the
// boundary entries and their places (kpos) in a launch before that of the inner entries, the two and this one, us: 9570 rows beside 23300
// boundary nodes 11.7 -> 6.3, 20011 beside 30011 14.6 -> 9.1, 29125 beside 197758 45.4 -> 37.1, 306250 beside 746157 53.0 -> 46.8, 578125
// beside 3.1 M 68.0 -> 64.4.  Every workgroup adds up the counts of all tiles before its own, which grows with the square of the partition and is not
// felt yet where a device is full: 63 M inner entries and 45 M boundary entries 610 -> 500, 75 M 986 -> 747.
__global__ void __launch_bounds__(kBdThreads) build_kernel(const BuildArgs a) {
  int block = blockIdx.x;
  if (block < a.list_blocks) return kept_rows_fill(a, block, a.list_blocks);
  block -= a.list_blocks;
  if (block < a.bd_tiles) return bd_fill_tile(a, block);
  block -= a.bd_tiles;
  if (block < a.row_blocks) return row_starts(a, block);
  block -= a.row_blocks;
  if (block < a.entry_blocks) return inner_entries(a, block);
  copy_static<kBdThreads>(a.st, a.n_in, a.e_in, block - a.entry_blocks, a.copy_blocks);
}

hipError_t build_subgraph(const SubgraphBuild &g, bool counted, hipStream_t s) {
  hipError_t e = hipSuccess;
  const int tiles = scan_tiles(g.bd.e_bd);
  if (tiles > 0 && !counted) {
    bd_count_kernel<<<tiles, kBdThreads, 0, s>>>(g.bd, g.ballots);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // eight lanes per list, for as many lists as there may be: beyond this many workgroups, most of which would find no
  // kept node left, each one takes several
  const int list_blocks = (int)std::min<int64_t>(((int64_t)g.n_halo + kListsPerBlock - 1) / kListsPerBlock, 4096);
  BuildArgs a{};
  a.n_in = g.n_in;
  a.e_in = g.e_in;
  a.inner_ptr = g.sp.inner_ptr; a.bd_ptr = g.sp.bd_ptr; a.in_col = g.sp.in_col; a.in_bdp = g.sp.in_bdp;
  a.row_ptr = g.row_ptr; a.nnz = g.nnz;
  a.entry_blocks = (int)((g.e_in + kEntryTile - 1) / kEntryTile);
  a.row_blocks = g.n_in / kEntryTile + 1;
  a.bd = g.bd;
  a.bd_tiles = tiles;
  a.bd_row = g.sp.bd_row; a.remap = g.remap; a.col_idx = g.col_idx;
  a.n_kept = g.n_kept; a.kept_ids = g.kept_ids; a.halo_ptr = g.halo_ptr; a.halo_col = g.halo_col; a.kept_start = g.kept_start;
  a.t_tail_ptr = g.t_row_ptr + g.n_in; a.t_col_idx = g.t_col_idx;
  a.list_blocks = list_blocks;
  a.st = StaticRows{g.t_in_ptr, g.t_in_col, g.t_row_ptr, g.t_col_idx};
  a.copy_blocks = g.static_rows ? std::min(a.entry_blocks, 16384) : 0;
  build_kernel<<<list_blocks + tiles + a.row_blocks + a.entry_blocks + a.copy_blocks, kBdThreads, 0, s>>>(a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------- set-up
__global__ void __launch_bounds__(kThreads)
copy_static_kernel(const StaticRows st, int32_t n_in, int64_t e_in) {
  copy_static<kThreads>(st, n_in, e_in, blockIdx.x, gridDim.x);
}

hipError_t copy_static_rows(int32_t n_in, int64_t e_in, const int32_t *t_in_ptr, const int32_t *t_in_col,
                            int32_t *t_row_ptr, int32_t *t_col_idx, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>(((int64_t)n_in + 1 + e_in + 4 * kThreads - 1) / (4 * kThreads), 16384);
  copy_static_kernel<<<(unsigned)blocks, kThreads, 0, s>>>(StaticRows{t_in_ptr, t_in_col, t_row_ptr, t_col_idx}, n_in, e_in);
  return hipGetLastError();
}

}  // namespace bns
