// Selection step and subgraph step of Algorithm 1 for a small partition, in one launch.
//
// The general path spends three launches per epoch on these two steps, each a few microseconds long
// whatever the size; for a partition of some ten thousand entries that is a fifth to a third of the whole
// training step.  Here one workgroup of 1024 threads runs the same stages back to back, with a
// barrier where the general path has a kernel boundary.  What bounds it is the chain of dependent reads, so the static
// arrays are asked for at the start, whatever one stage leaves for the next stays in LDS (keep bits, prefixes, lengths, positions),
// and the barriers wait for LDS alone, not for the stores to
// memory (steps of 64-16-8, 2000 rows of 2.5 entries beside 4000 boundary nodes 41.9 -> 37.4 us, 1200 of 8 beside 2400 38.9 -> 35.6).
// Every output is an integer array with a unique value: both paths write the same bits.
#include "pack_device.hpp"
#include "small_device.hpp"

namespace bns {

namespace {

// Workgroup 0 does all of it; the others pack weights.
template <int NB, int NE>
__global__ void __launch_bounds__(kSmallThreads) sample_build_small_kernel(const SmallArgs a, const PackJobs pack) {
  if (blockIdx.x > 0) pack_unit(pack, (blockIdx.x - 1) * (kSmallThreads / kWave) + threadIdx.x / kWave);
  else sample_and_build<NB, NE>(a);
}

}  // namespace

bool sample_build_small_fits(int32_t n_in, int32_t n_halo, int64_t e_in, int64_t e_bd, int32_t expected_kept) {
  return n_halo <= kSmallMaxHalo && e_bd <= kSmallMaxBoundaryEntries &&
         e_in + 3 * (int64_t)n_in + n_halo + 12 * (int64_t)expected_kept <= kSmallMaxWork;
}

hipError_t sample_build_small(const SmallArgs &a, const PackJobs &jobs, hipStream_t s) {
  if (a.n_halo > kSmallMaxHalo || a.e_bd > kSmallMaxBoundaryEntries) return hipErrorInvalidValue;
  const int pack_blocks = (jobs.units + kSmallThreads / kWave - 1) / (kSmallThreads / kWave);
  // (ten replayed epochs, at the larger limits and so, us: 500 rows beside 330 boundary nodes 341 / 331, 900 beside 700 347 / 337, 400
  // beside 100 330 / 330; single steps within 1 us of each other, either way)
  if (a.n_halo <= kSmallThreads && a.e_bd <= kSmallThreads)
    sample_build_small_kernel<1, 1><<<1 + pack_blocks, kSmallThreads, 0, s>>>(a, jobs);
  else
    sample_build_small_kernel<kSmallMaxHalo / kSmallThreads, kSmallMaxBoundaryEntries / kSmallThreads><<<1 + pack_blocks, kSmallThreads, 0, s>>>(a, jobs);
  return hipGetLastError();
}

}  // namespace bns
