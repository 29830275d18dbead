// fp32 products on the bf16 matrix instruction, by three-way splitting (Henry, Tang, Heinecke: Leveraging the bfloat16
// artificial intelligence datatype for higher-precision computations, ARITH 2019).
//
// An fp32 value is the exact sum of three bf16 values: hi = bf16(x), mid = bf16(x - hi) and
// lo = x - hi - mid (both differences are exact, and 3 x 8 significand bits hold the 24 of x).  A
// product of two such sums needs six of its nine partial products: the three left out (mid lo,
// lo mid, lo lo) are below 2^-26 of the product, a quarter of the rounding that an fp32 sum makes
// at every step.  Each partial product is exact in fp32.
//
// The six instructions of a 32-deep step start from zero, smallest products first, so that only the last one rounds at
// the size of the step's sum; that sum is then added to the running one in fp32.  Error against fp64 (2-norm, normal
// operands), beside a chain of v_mfma_f32_32x32x2_f32 and beside one accumulator through all instructions:
//   dZ W^T, depth  64: 4.7e-8 (1.4e-7, 0.9e-7)   128: 5.7e-8 (2.0e-7, 1.5e-7)   512: 8.9e-8 (4.1e-7, 3.4e-7)
//   A^T dZ, 60000 rows of 128 x 128: 1.0e-7 (1.9e-7, 2.7e-7)   300000: 1.2e-7 (3.4e-7, 3.2e-7)
// The additions are free in gemm_rows; in gemm_tn they cost 4 to 8 % on tiles of 128 x 128.
// Below 2^-110 the lo piece, then the mid piece are subnormal: such an operand is held to an absolute 2^-134.  Forward results that may
// suffer from it are formed once more without a split (any_tiny).
//
// v_mfma_f32_16x16x32_bf16 runs at sixteen times the rate of the fp32 instruction, so six of them
// take 6/16 of its time.  Operands that are not finite, or round to an infinite hi (above 3.389e38), have no split:
// their results are formed once more without one.
#pragma once
#include <hip/hip_runtime.h>

#include "device_utils.hpp"

namespace bns {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // global memory takes any 4-byte alignment
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kFragBytes = 1024;             // one operand fragment: 64 lanes x 8 bf16 (16 rows x 32 k)
constexpr int kFragSet = 3 * kFragBytes;     // its three pieces

// The last piece of a row whose length is no multiple of 4 is read four floats from the end: behind a branch per element each
// read would wait for the one before.  row_end() makes of it the piece that starts at k, in a row of n >= 4 floats: moved down,
// zero past the end.
__device__ __forceinline__ int piece_start(int k, int n) { return min(k, n - 4); }
__device__ __forceinline__ f32x4 row_end(const f32x4 &x, int k, int n) {
  const int by = k - piece_start(k, n);
  const bool one = by & 1, two = by & 2, all = by >= 4;
  f32x4 y;
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = one ? (e < 3 ? x[e + 1 < 4 ? e + 1 : 3] : 0.f) : x[e];
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = two ? (e < 2 ? y[e + 2 < 4 ? e + 2 : 3] : 0.f) : y[e];
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = all ? 0.f : y[e];
  return y;
}

// The pieces of two values, packed in pairs (first value in the low half).
__device__ __forceinline__ void split_pair(float x, float y, unsigned &hi, unsigned &mid, unsigned &lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){x, y}, bf16x2));
  const float rx = x - __builtin_bit_cast(float, hi << 16), ry = y - __builtin_bit_cast(float, hi & 0xffff0000u);
  mid = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){rx, ry}, bf16x2));
  const float sx = rx - __builtin_bit_cast(float, mid << 16), sy = ry - __builtin_bit_cast(float, mid & 0xffff0000u);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){sx, sy}, bf16x2));
}

struct Frag3 { bf16x8 p[3]; };  // hi, mid, lo of 8 values

// NEG: the pieces of the negated values.
template <bool NEG = false>
__device__ __forceinline__ Frag3 split8(const f32x4 &a_in, const f32x4 &b_in) {
    const f32x4 a = NEG ? -a_in : a_in, b = NEG ? -b_in : b_in;
  u32x4 h, m, l;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    unsigned x, y, z;
    split_pair(a[2 * i], a[2 * i + 1], x, y, z);
    h[i] = x; m[i] = y; l[i] = z;
    split_pair(b[2 * i], b[2 * i + 1], x, y, z);
    h[2 + i] = x; m[2 + i] = y; l[2 + i] = z;
  }
  Frag3 f;
  f.p[0] = __builtin_bit_cast(bf16x8, h);
  f.p[1] = __builtin_bit_cast(bf16x8, m);
  f.p[2] = __builtin_bit_cast(bf16x8, l);
  return f;
}

// t[r] = x . y[r] for R second operands, smallest partial products first; the results are taken in
// turn so that consecutive instructions do not wait for each other.  The instruction cuts off what an addend has below
// the last bit of the sum, downwards.  So that these cuts do not add up to a bias, half of the sums run on a
// negated operand and are negated at the end: every other column tile of gemm_rows, every other split of gemm_tn.
template <int R>
__device__ __forceinline__ void mfma_split(f32x4 (&t)[R], const Frag3 &x, const Frag3 (&y)[R]) {
  constexpr int px[6] = {0, 2, 1, 0, 1, 0}, py[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
  for (int r = 0; r < R; ++r) t[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int r = 0; r < R; ++r)
      t[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.p[px[i]], y[r].p[py[i]], t[r], 0, 0, 0);
}

// An infinite operand has no split (its other pieces are NaN), nor has one beyond 3.389e38, which rounds to an infinite
// piece, and a product near the top of the range can overflow in its first piece alone.  All of these end in a result that
// is not finite, and such a result is formed once more as the plain fp32 sum, so that infinities and NaN come out as from the operands
// themselves.  Looking costs an instruction per result and tile; a product all of whose results are NaN takes some 50 to 80
// times as long (89625 x 512 x 512: 11 and 20 ms), one infinite element a few times.
__device__ __forceinline__ float nonfinite_seed(float z, const f32x4 &v) {  // z stays 0 while all values are finite
#pragma unroll
  for (int e = 0; e < 4; ++e) z = fmaf(v[e], 0.f, z);
  return z;
}
// Any of the values other than zero and below 2^-64?  Operands below 2^-110 have pieces below the bf16 range and are held to an absolute
// 2^-134.  A result that feels it is small itself, unless it has operands above 2^30 on the other side (2^-134 of 1024 terms against 2^-24 of
// 2^-64).  Dead rows and columns are exactly zero and pass.  Looking costs nothing that could be measured (578125 rows, 256 -> 172).
__device__ __forceinline__ bool any_tiny(const f32x4 &v) {
  unsigned least = ~0u;  // of twice the bits less one: zeros count as the largest
#pragma unroll
  for (int e = 0; e < 4; ++e) least = min(least, (__float_as_uint(v[e]) << 1) - 1u);
  return least < (__float_as_uint(0x1p-64f) << 1) - 1u;
}
__device__ __forceinline__ bool is_finite(float x) { return fabsf(x) <= 3.40282347e38f; }

// One 16-byte-per-lane copy from global memory straight into LDS (lane i lands at lds + 16 i; both
// arguments as the whole wavefront sees them).  Written as assembly so that the compiler does not
// wait for it before unrelated LDS reads: the caller waits with lds_dma_wait() and a barrier.  It overwrites M0, which
// the compiler reserves (it says so when the register is named) but would otherwise take for unchanged.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma16(const void *src_lane, unsigned lds_offset) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src_lane), "s"(lds_offset) : "m0", "memory");
}
#pragma clang diagnostic pop
__device__ __forceinline__ void lds_dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ unsigned lds_offset_of(const void *p) {  // LDS pointers: the low half of the generic address
  return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)p);
}

}  // namespace bns
