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
//   kpos[k]     = kept boundary entries before boundary entry k            (prefix sum)
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

struct FillArgs {
  // kept boundary entries of the sampled CSR
  int32_t n_in;
  BdCount bd;
  int bd_tiles;
  const int32_t *bd_row, *remap, *inner_ptr;
  int32_t *kpos, *col_idx;
  // rows of the kept boundary nodes in the transposed CSR
  const int32_t *n_kept, *kept_ids, *halo_ptr, *halo_col, *kept_start;
  int32_t *t_tail_ptr, *t_col_idx;
};

// Positions of a tile's boundary entries, from the keep flags: those inside a pass come from the population count of
// the lower lanes' bits.  A kept entry also gets its place in col_idx; the 4-byte rank is only fetched for those.
__device__ __forceinline__ void bd_fill_tile(const FillArgs &a) {
  __shared__ int wave_cnt[kBdWaves];
  const int lane = lane_id(), wid = threadIdx.x / kWave;
  const int64_t e_bd = a.bd.e_bd;
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)wid * (kBdPasses * kWave);
  unsigned long long mask[kBdPasses];
  int cnt = 0;
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i) {
    mask[i] = base + i * kWave < e_bd ? a.bd.mask[(base >> 6) + i] : 0ull;
    cnt += __popcll(mask[i]);
  }
  if (lane == 0) wave_cnt[wid] = cnt;
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
  tiles_before<kBdThreads, 1>(a.bd.sums, blockIdx.x, a.bd_tiles, false, before, total);
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i)
    if ((mask[i] >> lane) & 1ull) {
      node[i] = a.n_in + a.remap[node[i]];
      row[i] = a.inner_ptr[row[i] + 1];
    }
  int run = before[0];
  for (int w = 0; w < wid; ++w) run += wave_cnt[w];
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i) {
    const int64_t k = base + i * kWave + lane;
    const bool kept = (mask[i] >> lane) & 1ull;
    const int pos = run + __popcll(mask[i] & lower);
    if (k < e_bd) {
      a.kpos[k] = pos;
      if (kept) a.col_idx[row[i] + pos] = node[i];
      if (k == e_bd - 1) a.kpos[e_bd] = pos + (kept ? 1 : 0);
    }
    run += __popcll(mask[i]);
  }
}

// Rows of the kept boundary nodes in the transposed CSR: kept node r (boundary node b =
// kept_ids[r]) gets b's static list of inner neighbours.  Where each row starts was settled by the
// sampler (a prefix sum of the list lengths in kept order, kept_start[0..n_kept]); eight lanes copy
// one list and write the row's start.  The lists that are too long for eight lanes are left to the whole workgroup
// (197 758 boundary nodes with up to 5 800 neighbours: 81 us with eight lanes for each list, now 16).
constexpr int kLongList = 256;
constexpr int kListsPerBlock = kBdThreads / 8;
__device__ __forceinline__ void kept_rows_fill(const FillArgs &a, int block, int n_blocks) {
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

__global__ void __launch_bounds__(kBdThreads) fill_kernel(const FillArgs a) {
  if ((int)blockIdx.x < a.bd_tiles) bd_fill_tile(a);
  else kept_rows_fill(a, blockIdx.x - a.bd_tiles, gridDim.x - a.bd_tiles);
}

// Row starts and the inner entries in one launch: both follow in closed form from kpos (row v's
// entries move down by the kept boundary entries of the rows before it, kpos[bd_ptr[v]]; every
// inner entry carries its row's bd_ptr, so it needs one gather).
// The workgroups from `blocks` on copy the rows of the inner nodes in the transposed CSR, which never change (the
// transpose of the inner-inner block), where the destination does not hold them yet.
struct StaticRows {
  const int32_t *ptr, *col;
  int32_t *t_row_ptr, *t_col_idx;
};

__device__ __forceinline__ void copy_static(const StaticRows &st, int32_t n_in, int64_t e_in, int block, int n_blocks) {
  for (int64_t i = (int64_t)block * kThreads + threadIdx.x; i < n_in + 1 + e_in; i += (int64_t)n_blocks * kThreads) {
    if (i <= n_in) st.t_row_ptr[i] = st.ptr[i];
    else st.t_col_idx[i - n_in - 1] = st.col[i - n_in - 1];
  }
}

constexpr int kFinishPasses = 8, kFinishTile = kFinishPasses * kThreads;

__global__ void __launch_bounds__(kThreads)
finish_csr_kernel(int32_t n_in, int64_t e_in, int64_t e_bd, const int32_t *__restrict__ inner_ptr,
                  const int32_t *__restrict__ bd_ptr, const int32_t *__restrict__ kpos,
                  const int32_t *__restrict__ in_col, const int32_t *__restrict__ in_bdp,
                  int32_t *__restrict__ row_ptr, int32_t *__restrict__ col_idx, int32_t *__restrict__ nnz, int blocks,
                  const StaticRows st) {
  if ((int)blockIdx.x >= blocks) {
    copy_static(st, n_in, e_in, blockIdx.x - blocks, gridDim.x - blocks);
    return;
  }
  // a tile of kFinishTile entries per workgroup and its reads all at once: they hang on each other (in_bdp, kpos, place)
  const int64_t j0 = (int64_t)blockIdx.x * kFinishTile + threadIdx.x;
  int c[kFinishPasses], k[kFinishPasses];
#pragma unroll
  for (int i = 0; i < kFinishPasses; ++i) {
    const int64_t j = j0 + i * kThreads;
    c[i] = j < e_in ? in_col[j] : 0;
    k[i] = j < e_in && e_bd > 0 ? in_bdp[j] : -1;
  }
  const int64_t stride = (int64_t)blocks * kThreads;
  const int64_t t0 = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  for (int64_t v = t0; v <= n_in; v += stride) {
    const int r = inner_ptr[v] + (e_bd > 0 ? kpos[bd_ptr[v]] : 0);
    row_ptr[v] = r;
    if (v == n_in) *nnz = r;
  }
#pragma unroll
  for (int i = 0; i < kFinishPasses; ++i) k[i] = k[i] >= 0 ? kpos[k[i]] : 0;
#pragma unroll
  for (int i = 0; i < kFinishPasses; ++i)
    if (j0 + i * kThreads < e_in) col_idx[j0 + i * kThreads + k[i]] = c[i];
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
  if (tiles + list_blocks > 0) {
    FillArgs a{};
    a.n_in = g.n_in;
    a.bd = g.bd;
    a.bd_tiles = tiles;
    a.bd_row = g.sp.bd_row; a.remap = g.remap; a.inner_ptr = g.sp.inner_ptr;
    a.kpos = g.kpos; a.col_idx = g.col_idx;
    a.n_kept = g.n_kept; a.kept_ids = g.kept_ids; a.halo_ptr = g.halo_ptr; a.halo_col = g.halo_col; a.kept_start = g.kept_start;
    a.t_tail_ptr = g.t_row_ptr + g.n_in; a.t_col_idx = g.t_col_idx;
    fill_kernel<<<tiles + list_blocks, kBdThreads, 0, s>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int64_t work = std::max<int64_t>(g.e_in, (int64_t)g.n_in + 1);
  const int blocks = (int)((work + kFinishTile - 1) / kFinishTile);
  const int copy = g.static_rows ? std::min(blocks, 16384) : 0;
  finish_csr_kernel<<<blocks + copy, kThreads, 0, s>>>(g.n_in, g.e_in, g.bd.e_bd, g.sp.inner_ptr, g.sp.bd_ptr, g.kpos,
                                                       g.sp.in_col, g.sp.in_bdp, g.row_ptr, g.col_idx, g.nnz, blocks,
                                                       StaticRows{g.t_in_ptr, g.t_in_col, g.t_row_ptr, g.t_col_idx});
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------- set-up
__global__ void __launch_bounds__(kThreads)
copy_static_kernel(const StaticRows st, int32_t n_in, int64_t e_in) {
  copy_static(st, n_in, e_in, blockIdx.x, gridDim.x);
}

hipError_t copy_static_rows(int32_t n_in, int64_t e_in, const int32_t *t_in_ptr, const int32_t *t_in_col,
                            int32_t *t_row_ptr, int32_t *t_col_idx, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>(((int64_t)n_in + 1 + e_in + 4 * kThreads - 1) / (4 * kThreads), 16384);
  copy_static_kernel<<<(unsigned)blocks, kThreads, 0, s>>>(StaticRows{t_in_ptr, t_in_col, t_row_ptr, t_col_idx}, n_in, e_in);
  return hipGetLastError();
}

}  // namespace bns
