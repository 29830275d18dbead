// Boundary-node sampling (Algorithm 1, selection step): every boundary node is kept
// independently with probability p, decided by a counter-based draw so that the decision
// depends only on (seed, epoch, partition, global node id).  Kept nodes are compacted in
// ascending order with wavefront ballots and prefix sums.
#include "build_device.hpp"
#include "pack_device.hpp"

namespace bns {

// First output word of the Philox draw.
__device__ __forceinline__ uint32_t philox4x32_10_word0(uint32_t c0, uint32_t c1, uint32_t c2,
                                                        uint32_t c3, uint32_t k0, uint32_t k1) {
  philox4x32_10(c0, c1, c2, c3, k0, k1);
  return c0;
}

constexpr int kSampleThreads = kBdThreads;  // one launch carries both
constexpr int kSampleIters = kScanTile / kSampleThreads;  // passes over a tile
constexpr int kWordsPerTile = kScanTile / kWave;          // 32

// Pass 1: keep flags as one 64-bit ballot word per 64 consecutive boundary nodes, and the
// number of kept nodes per tile (tile_sums[tile], raw counts).  With halo_ptr (the boundary
// nodes' static lists of inner neighbours) also the summed list length of the tile's kept nodes
// (tile_sums[tiles + tile]): the rows of the kept nodes in the transposed subgraph are laid out in
// kept order, so their starts are a prefix sum of exactly these lengths.
__global__ void __launch_bounds__(kSampleThreads)
sample_flags_kernel(const int64_t *__restrict__ halo_gid, int32_t n_halo, uint32_t k0, uint32_t k1,
                    uint32_t epoch, const uint32_t *__restrict__ epoch_dev, uint32_t part_id,
                    uint64_t threshold, const int32_t *__restrict__ halo_ptr, uint64_t *__restrict__ ballots,
                    int32_t *__restrict__ tile_sums, int tiles, const PackJobs pack) {
  if ((int)blockIdx.x >= tiles) {
    pack_unit(pack, (blockIdx.x - tiles) * (kSampleThreads / kWave) + threadIdx.x / kWave);
    return;
  }
  if (epoch_dev) epoch = *epoch_dev;  // epoch counter kept on the device (graph replay)
  const int lane = lane_id();
  int cnt = 0, len = 0;
  uint64_t gid[kSampleIters];
  bool keep[kSampleIters];
#pragma unroll
  for (int it = 0; it < kSampleIters; ++it) {
    const int64_t b = (int64_t)blockIdx.x * kScanTile + it * kSampleThreads + threadIdx.x;
    gid[it] = b < n_halo ? (uint64_t)halo_gid[b] : 0;
  }
#pragma unroll
  for (int it = 0; it < kSampleIters; ++it) {
    const int64_t b = (int64_t)blockIdx.x * kScanTile + it * kSampleThreads + threadIdx.x;
    const uint32_t u = philox4x32_10_word0((uint32_t)gid[it], (uint32_t)(gid[it] >> 32), epoch, part_id, k0, k1);
    keep[it] = b < n_halo && (uint64_t)u < threshold;
    const uint64_t word = __ballot(keep[it]);
    if (lane == 0 && b < n_halo) ballots[b >> 6] = word;
    cnt += (lane == 0) ? __popcll(word) : 0;
  }
  if (halo_ptr) {
    int end[kSampleIters], begin[kSampleIters];
#pragma unroll
    for (int it = 0; it < kSampleIters; ++it) {
      const int64_t b = (int64_t)blockIdx.x * kScanTile + it * kSampleThreads + threadIdx.x;
      begin[it] = keep[it] ? halo_ptr[b] : 0;
      end[it] = keep[it] ? halo_ptr[b + 1] : 0;
    }
#pragma unroll
    for (int it = 0; it < kSampleIters; ++it) len += end[it] - begin[it];
  }
  __shared__ int red[2][kSampleThreads / kWave];
  cnt = wave_sum(cnt);
  len = wave_sum(len);
  if (lane == 0) {
    red[0][threadIdx.x / kWave] = cnt;
    red[1][threadIdx.x / kWave] = len;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int total = 0, len_total = 0;
#pragma unroll
    for (int w = 0; w < kSampleThreads / kWave; ++w) {
      total += red[0][w];
      len_total += red[1][w];
    }
    tile_sums[blockIdx.x] = total;
    if (halo_ptr) tile_sums[tiles + blockIdx.x] = len_total;
  }
}

// Pass 2: rank of every kept node = kept nodes in earlier tiles (summed by the block itself) +
// kept nodes in earlier words of the tile + kept lanes below it in its own word.  The tile's kept
// nodes are first compacted into LDS in rank order; the block then walks the ranks, so that
// kept_ids is written with consecutive addresses and (with halo_ptr) the start of each kept node's
// row in the transposed subgraph, first + the list lengths of the kept nodes before it, comes from a
// block scan over just the kept ones: kept_start[rank], and kept_start[n_kept] = the end.  With rec, the
// record that the forward aggregates read per kept node (its boundary index and weight) goes with it.
// Block 0 also writes the totals.  The blocks from `tiles` on count the kept boundary entries, which needs the keep
// bits alone.
__global__ void __launch_bounds__(kSampleThreads)
sample_write_kernel(int32_t n_halo, const uint64_t *__restrict__ ballots,
                    const int32_t *__restrict__ tile_counts, int32_t *__restrict__ kept_ids,
                    int32_t *__restrict__ remap, int32_t *__restrict__ n_kept,
                    const int32_t *__restrict__ halo_ptr, int32_t first, int32_t *__restrict__ kept_start,
                    int2 *__restrict__ rec, const float *__restrict__ dis_halo, float s_halo, int tiles, const BdCount count) {
  if ((int)blockIdx.x >= tiles) {
    bd_count_tile(count, ballots, blockIdx.x - tiles);
    return;
  }
  __shared__ int word_prefix[kWordsPerTile + 1];
  __shared__ int kept_b[kScanTile];
  const int lane = lane_id();
  __shared__ uint64_t words[kWordsPerTile];
  const int64_t word0 = (int64_t)blockIdx.x * kWordsPerTile;
  const int64_t n_words = ((int64_t)n_halo + kWave - 1) / kWave;
  if (threadIdx.x < kWave) {
    const int64_t w = word0 + threadIdx.x;
    const uint64_t word = threadIdx.x < kWordsPerTile && w < n_words ? ballots[w] : 0ull;
    const int c = __popcll(word);
    const int inc = wave_inclusive_scan(c);
    if (threadIdx.x < kWordsPerTile) {
      words[threadIdx.x] = word;
      word_prefix[threadIdx.x] = inc - c;
    }
    if (threadIdx.x == kWordsPerTile - 1) word_prefix[kWordsPerTile] = inc;  // kept nodes of the tile
  }
  // kept nodes and the length of their lists in the tiles before this one (ends with a barrier)
  int before[2], total[2];
  if (halo_ptr) {
    tiles_before<kSampleThreads, 2>(tile_counts, blockIdx.x, tiles, blockIdx.x == 0, before, total);
  } else {
    int b1[1], t1[1];
    tiles_before<kSampleThreads, 1>(tile_counts, blockIdx.x, tiles, blockIdx.x == 0, b1, t1);
    before[0] = b1[0];
    total[0] = t1[0];
    before[1] = total[1] = 0;
  }
  const int base = before[0];
  int run = first + before[1];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *n_kept = total[0];
    if (halo_ptr) kept_start[total[0]] = first + total[1];
  }
#pragma unroll
  for (int it = 0; it < kSampleIters; ++it) {
    const int local = it * kSampleThreads + threadIdx.x;
    const int64_t b = (int64_t)blockIdx.x * kScanTile + local;
    if (b < n_halo) {
      const uint64_t word = words[local >> 6];
      if ((word >> lane) & 1ull) {
        const int r = word_prefix[local >> 6] + __popcll(word & ((1ull << lane) - 1ull));
        kept_b[r] = (int32_t)b;
        remap[b] = base + r;
      } else {
        remap[b] = -1;
      }
    }
  }
  __syncthreads();
  const int tile_kept = word_prefix[kWordsPerTile];
  for (int r0 = 0; r0 < tile_kept; r0 += kSampleThreads) {  // block-uniform trip count
    const int r = r0 + threadIdx.x;
    const int b = r < tile_kept ? kept_b[r] : -1;
    int len = 0;
    float dis = 1.f;
    if (b >= 0) {
      if (halo_ptr) len = halo_ptr[b + 1] - halo_ptr[b];
      if (rec && dis_halo) dis = dis_halo[b];
    }
    if (b >= 0) {
      kept_ids[base + r] = b;
      if (rec) rec[base + r] = make_int2(b, __float_as_int(dis_halo ? s_halo * dis : s_halo));
    }
    if (halo_ptr) {
      int sum;
      const int before = block_exclusive_scan<kSampleThreads>(len, &sum);
      if (b >= 0) kept_start[base + r] = run + before;
      run += sum;
    }
  }
}

hipError_t sample_boundary(const int64_t *halo_gid, int32_t n_halo, uint64_t seed, uint32_t epoch,
                           const uint32_t *epoch_dev, uint32_t part_id, uint64_t threshold, uint64_t *ballots,
                           int32_t *tile_sums, int32_t *kept_ids, int32_t *remap, int32_t *n_kept,
                           const int32_t *halo_ptr, int32_t first, int32_t *kept_start, int2 *rec, const float *dis_halo, float s_halo,
                           const PackJobs *pack, const BdCount *count, hipStream_t s) {
  if (!kept_start) halo_ptr = nullptr;
  const int nb = scan_tiles(n_halo) > 0 ? scan_tiles(n_halo) : 1;
  const PackJobs jobs = pack ? *pack : PackJobs{};
  const int pack_blocks = (jobs.units + kSampleThreads / kWave - 1) / (kSampleThreads / kWave);
  sample_flags_kernel<<<nb + pack_blocks, kSampleThreads, 0, s>>>(halo_gid, n_halo, (uint32_t)seed,
                                                    (uint32_t)(seed >> 32), epoch, epoch_dev, part_id,
                                                    threshold, halo_ptr, ballots, tile_sums, nb, jobs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  sample_write_kernel<<<nb + (count ? scan_tiles(count->e_bd) : 0), kSampleThreads, 0, s>>>(n_halo, ballots, tile_sums, kept_ids, remap, n_kept,
                                                    halo_ptr, first, kept_start, rec, dis_halo, s_halo, nb, count ? *count : BdCount{});
  return hipGetLastError();
}

}  // namespace bns
