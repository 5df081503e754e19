// Floats as pairs of half-precision terms, for products of floats on the half-precision matrix cores.
//
// The matrix cores multiply f16 sixteen times as fast as float.  A float v, scaled by a power of two so that the
// largest magnitude under its scale lies in [2^14, 2^15), is hi + lo / 2^11 with hi = v rounded to f16 (11 significand
// bits, and the sign of the remainder is a twelfth) and lo = the remainder times 2^11 rounded to f16: 23 bits, one short
// of a float's significand (a quarter of all floats lose their last bit, an error of at most 2^-23 of the element).  Of the
// four term products hi*hi, hi*lo, lo*hi and lo*lo the last, at most 2^-22 of the product and 2^-24.6 on average, is left
// out.  hi*hi is added in one accumulator, the two mixed products in another, which joins the first with its factor 2^-11
// at the end: the large accumulator is rounded once per 16 contraction elements (v_mfma_f32_32x32x16_f16), where the
// float instruction rounds it once per two, so the sums of ordinary data come out no further from the exact ones.
//
// Range.  One operand (the activations, or the gradient of them) has a scale per image, so that an image's results do not
// depend on the images beside it; the kernel matrix has one, and so has either operand of the kernel gradient, whose sums
// run over the images.  Under its scale an element keeps the 23 bits down to 2^-27 of the largest one and an absolute
// error of 2^-36 (2^-50 of the largest) below that.  The re-laying passes count the elements they cannot keep to 21 bits
// (below 2^-15 scaled); where they exceed one in 8192 (or 1024 in all), or where an element is not finite, the product is
// DECLINED: its blocks leave at once and the float kernel, enqueued behind it and otherwise leaving at once itself, computes
// the image (any declined element of the kernel matrix or of a kernel gradient: all of it).  The decision stays on the
// device.  So rare small elements - one in 10^8 of normally distributed ones - cost nothing, and an operand whose elements
// span more than the terms hold gives what the float kernel gives, in that kernel's time and the re-laying's (64 64 64 64 ->
// 32 5 5 forward 0.33 ms against 0.28 in float and 0.15 in two terms, all in parts of the batch).  An infinity would meet
// terms that are zero where the float is not, and the zeros that pad a tile.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace vcnn {

static constexpr uint32_t kNotLookedAt = 2;
static constexpr int kAbsMaxBlocks = 512;  // partial maxima of an operand with one scale

// What a two-term product keeps about its two operands in the workspace (device pointers; the host lays them out).
struct SplitScales {
  uint32_t* partial[2];  // largest magnitude (float bits) of each scanning block's share
  int32_t* exponent[2];  // scaled by 2^exponent: one per image, one
  uint32_t* small[2];    // elements below 2^-15 when scaled: per image, one
  uint32_t* any;         // the words of Declined: kNotLookedAt in `any` and `image` keeps the product from images that `only`
  uint32_t* all;         // leaves out, so that its kernels need to look at nothing more
  uint32_t* image;
  uint32_t limit[2];     // more small elements than this decline
  int blocks;            // scanning blocks per image of operand 0
  Declined only;         // (of_any, of) the images that the product is for

  Declined declined() const { return {any, all, image, only.of_any, only.of}; }
  // The same for images n0 and on (a part of the batch).
  SplitScales from(int n0) const {
    SplitScales s = *this;
    s.exponent[0] += n0, s.small[0] += n0, s.image += n0, s.only = s.only.from(n0);
    return s;
  }
};

// The largest of `blocks` partial maxima; called by all 256 threads of a block.
__device__ __forceinline__ uint32_t split_max(const uint32_t* partial, int blocks) {
  __shared__ uint32_t wave_max[4];
  const int tid = threadIdx.x;
  uint32_t m = 0;
  for (int i = tid; i < blocks; i += 256) m = max(m, partial[i]);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
  if ((tid & 63) == 0) wave_max[tid >> 6] = m;
  __syncthreads();
  return max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
}
// The exponent for a largest magnitude (a denormal one counts as 2^-126; zeros, and what is not finite, need no scale).
__device__ __forceinline__ int split_exponent(uint32_t largest) {
  return largest == 0 || largest >= 0x7f800000u ? 0 : 14 - (max((int)(largest >> 23), 1) - 127);
}
__device__ __forceinline__ void decline(const SplitScales& sc, int operand, int image) {
  *sc.any = 1;
  if (operand == 0) sc.image[image] = 1;
  else *sc.all = 1;
}
// One thread per scale: leaves it for the product, and declines what holds an element that is not finite.
__device__ __forceinline__ void note_scale(const SplitScales& sc, int operand, int image, uint32_t largest) {
  sc.exponent[operand][operand == 0 ? image : 0] = split_exponent(largest);
  if (largest >= 0x7f800000u) decline(sc, operand, image);
}
// Adds a thread's count of small elements; called by whole blocks of 256.  A block that has none, as on ordinary data,
// touches nothing; one that exceeds the limit by itself says so without the shared counter, whose atomics come one after
// the other (all of 64 64 64 64 small: with an atomic per wave the scan and the re-laying took 340 us instead of 60).
__device__ __forceinline__ void note_small(const SplitScales& sc, int operand, int image, int count) {
  if (!__syncthreads_or(count)) return;
  __shared__ int waves[4];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) count += __shfl_xor(count, d);
  if ((threadIdx.x & 63) == 0) waves[threadIdx.x >> 6] = count;
  __syncthreads();
  if (threadIdx.x != 0) return;
  const uint32_t sum = (uint32_t)(waves[0] + waves[1] + waves[2] + waves[3]), limit = sc.limit[operand];
  uint32_t* const total = sc.small[operand] + (operand == 0 ? image : 0);
  if (sum > limit) return decline(sc, operand, image);
  // (past the limit already: a read in place of the atomic, a tenth of its time)
  if (__hip_atomic_load(total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > limit) return;
  if (atomicAdd(total, sum) + sum > limit) decline(sc, operand, image);
}

// Finds the elements below 2^-15 when scaled.  key(): the magnitude's bits, zero (exact at any scale) above all others;
// the splitting passes keep the least key of a thread's elements, two instructions for one, and count where it is below
// the limit.
struct SmallElements {
  uint32_t limit, least;
  __device__ __forceinline__ explicit SmallElements(int exponent) : least(~0u) {
    const uint32_t bound = __float_as_uint(ldexpf(1.f, -15 - exponent));  // (0: no float is that small)
    limit = bound ? 2 * bound - 1 : 0;
  }
  static __device__ __forceinline__ uint32_t key(float v) { return (__float_as_uint(v) << 1) - 1u; }
  __device__ __forceinline__ void take(float v) { least = min(least, key(v)); }
  template <int N>
  __device__ __forceinline__ int count(const float (&v)[N]) const {
    int c = 0;
    if (least < limit) {
#pragma unroll
      for (int i = 0; i < N; ++i) c += key(v[i]) < limit;
    }
    return c;
  }
};

// The two terms of v * 2^exponent (v finite) as f16 bits: hi in the low half of the result, lo in the high half.
__device__ __forceinline__ uint32_t split_f16(float v, int exponent) {
  const float t = ldexpf(v, exponent);
  const _Float16 hi = (_Float16)t;
  const _Float16 lo = (_Float16)((t - (float)hi) * 2048.f);
  return (uint32_t)__builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
}
// The joined sum, still scaled.
__device__ __forceinline__ float join_f16(float hi, float lo) {
  return fmaf(lo, 1.f / 2048.f, hi);
}
// Eight split elements as one 16-byte word per term.
__device__ __forceinline__ void pack_terms(const uint32_t (&v)[8], uint4* hi, uint4* lo) {
  *hi = make_uint4((v[0] & 0xffffu) | v[1] << 16, (v[2] & 0xffffu) | v[3] << 16, (v[4] & 0xffffu) | v[5] << 16,
                   (v[6] & 0xffffu) | v[7] << 16);
  *lo = make_uint4(v[0] >> 16 | (v[1] & 0xffff0000u), v[2] >> 16 | (v[3] & 0xffff0000u), v[4] >> 16 | (v[5] & 0xffff0000u),
                   v[6] >> 16 | (v[7] & 0xffff0000u));
}

}  // namespace vcnn
