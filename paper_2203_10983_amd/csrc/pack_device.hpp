// Weight matrices as operand fragments, 1 KB each (64 lanes x 16 bytes), zero outside the matrix:
//   split: of W [N, K] transposed (fwd: of W [K, N] as it is), for gemm_rows.  For depth step s of 32 and column tile t of 16, at
//     ((s * tiles + t) * 3 + piece) KB, lane l's 8 values are column 16 t + l % 16 at the depths
//     32 s + 16 (e / 4) + 4 (l / 16) + e % 4, e = 0..7, negated in odd tiles (mfma_split)
//   fp32: of W [K, N], for gemm_rows_f32.  For depth step s of 32, column tile t of 32 and depth group j of 8, at
//     ((s * tiles + t) * 4 + j) KB, lane l's 4 values are column 32 t + l % 32 at the depths
//     32 s + 8 j + 2 i + l / 32, i = 0..3
#pragma once
#include "kernels.hpp"
#include "split_bf16.hpp"

namespace bns {

__host__ __device__ inline int k_steps(int K) { return (K + 31) / 32; }
__host__ __device__ inline int col_tiles(int N) { return (N + 15) / 16; }

// One wavefront packs unit u of the jobs: one depth step of one column tile.  Its elements are read without a branch between them, behind
// which each would wait for the one before (packing of 602 x 130 beside 15000 records, both forms: 9.4 -> 4.7 us).
__device__ __forceinline__ void pack_unit(const PackJobs &jobs, int u) {
  int q = 0;
  for (; q < jobs.n; ++q) {
    const int units = pack_units(jobs.j[q]);
    if (u < units) break;
    u -= units;
  }
  if (q == jobs.n) return;
  const PackJob &job = jobs.j[q];
  const int lane = lane_id();
  if (job.split) {
    const int T = col_tiles(job.N), s = u / T, t = u % T;
    const int n = t * 16 + (lane & 15), g = lane >> 4;
    f32x4 v[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = s * 32 + j * 16 + g * 4 + e;
        v[j][e] = job.W[(size_t)min(n, job.N - 1) * (job.fwd ? 1 : job.K) + (size_t)min(k, job.K - 1) * (job.fwd ? job.N : 1)];
      }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[j][e] = s * 32 + j * 16 + g * 4 + e < job.K && n < job.N ? v[j][e] : 0.f;
    const Frag3 f = t & 1 ? split8<true>(v[0], v[1]) : split8(v[0], v[1]);
    char *out = static_cast<char *>(job.out) + (size_t)u * kFragSet + lane * 16;
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<bf16x8 *>(out + p * kFragBytes) = f.p[p];
  } else {
    const int T = (job.N + 31) / 32, s = u / T, t = u % T;
    const int n = t * 32 + (lane & 31);
    char *out = static_cast<char *>(job.out) + (size_t)u * 4096 + lane * 16;
    f32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        v[j][i] = job.W[(size_t)min(s * 32 + j * 8 + i * 2 + (lane >> 5), job.K - 1) * job.N + min(n, job.N - 1)];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[j][i] = s * 32 + j * 8 + i * 2 + (lane >> 5) < job.K && n < job.N ? v[j][i] : 0.f;
      *reinterpret_cast<f32x4 *>(out + j * 1024) = v[j];
    }
  }
}

}  // namespace bns
