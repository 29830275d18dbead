// Device code of the subgraph step that more than one launch carries: the keep flags of a tile of boundary entries.
#pragma once
#include "device_utils.hpp"
#include "kernels.hpp"

namespace bns {

// A tile of kScanTile boundary entries per workgroup (the keep decision of a boundary node is one bit of the sampler's ballot
// words, a table of n_halo/8 bytes that stays in L2); every wavefront owns a contiguous piece of
// it and walks the piece 64 entries at a time.  The keep flags of a pass are one ballot word, written out for the
// pass over the same tile that places the entries; the number of kept entries per tile goes to sums.
// 512 threads a tile, and in every pass the reads of one stage all at once (they hang on each other: node, keep bit, rank, place):
// what these launches take is a few chains of reads.  When there were four in a training step, with 256 threads that went through a tile
// entry by entry / with 1024 / so, us: 9570 rows beside 23300 boundary nodes 28 / 24 / 25, 29125 beside 197758 (all kept) 97 / 87 / 86,
// 306250 beside 746157 75 / 73 / 70, 578125 beside 3.1 M 115 / 121 / 108.
constexpr int kBdThreads = 512;
constexpr int kBdWaves = kBdThreads / kWave;
constexpr int kBdPasses = kScanTile / kBdThreads;  // passes of 64 entries per wavefront

__device__ __forceinline__ void bd_count_tile(const BdCount &c, const uint64_t *__restrict__ ballots, int tile) {
  __shared__ int wave_cnt[kBdWaves];
  const int lane = lane_id(), wid = threadIdx.x / kWave;
  const int64_t base = (int64_t)tile * kScanTile + (int64_t)wid * (kBdPasses * kWave);
  int b[kBdPasses];
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i) {
    const int64_t k = base + i * kWave + lane;
    b[i] = k < c.e_bd ? c.bd_b[k] : -1;
  }
  uint64_t bits[kBdPasses];
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i) bits[i] = b[i] >= 0 ? ballots[b[i] >> 6] : 0ull;
  int cnt = 0, before[kBdPasses];
#pragma unroll
  for (int i = 0; i < kBdPasses; ++i) {
    const unsigned long long word = __ballot((bits[i] >> (b[i] & 63)) & 1ull);
    if (lane == 0 && base + i * kWave < c.e_bd) c.mask[(base >> 6) + i] = word;
    before[i] = cnt;
    cnt += __popcll(word);
  }
  if (lane == 0) wave_cnt[wid] = cnt;
  __syncthreads();
  if (lane == 0) {
    int run = 0;
    for (int w = 0; w < wid; ++w) run += wave_cnt[w];
#pragma unroll
    for (int i = 0; i < kBdPasses; ++i)
      if (base + i * kWave < c.e_bd) c.before[(base >> 6) + i] = run + before[i];
  }
  if (threadIdx.x == 0) {
    int total = 0;
#pragma unroll
    for (int w = 0; w < kBdWaves; ++w) total += wave_cnt[w];
    c.sums[tile] = total;
  }
}

}  // namespace bns
