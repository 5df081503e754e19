// Floats as pairs of half-precision terms, for products of floats on the half-precision matrix cores.
//
// The matrix cores multiply f16 sixteen times as fast as float.  A float v, scaled by a power of two so that the
// largest magnitude of its tensor lies in [2^14, 2^15), is hi + lo / 2^11 with hi = v rounded to f16 (11 significand
// bits, and the sign of the remainder is a twelfth) and lo = the remainder times 2^11 rounded to f16: 24 bits, the
// significand of a float, as long as |v| is above 2^-29 of the tensor's largest element; below that the remainder's
// error stays under 2^-50 of the largest element.  Of the four term products hi*hi, hi*lo, lo*hi and lo*lo the last
// lies below 2^-24 of the product - the rounding a float product has anyway - and is left out.  hi*hi is added in one
// accumulator, the two mixed products in another, which joins the first with its factor 2^-11 at the end: the large
// accumulator is rounded once per 16 contraction elements (v_mfma_f32_32x32x16_f16), where the float instruction
// rounds it once per two, so the sums come out closer to the exact ones than the float instruction's.
//
// Infinities and NaN: hi carries them (lo = 0), and the joined sum is hi's alone when that is not finite, so a
// non-finite element reaches exactly the sums it is part of.  The scale is taken from the finite elements.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vcnn {

static constexpr int kAbsMaxBlocks = 512;  // partial maxima per tensor

// what a split product keeps about its two operands in the workspace
struct SplitScales {
  uint32_t partial[2][kAbsMaxBlocks];  // largest finite magnitude of each block's share (float bits)
  int32_t exponent[2];                 // operand t was scaled by 2^exponent[t]
};
static constexpr size_t kSplitScalesBytes = (sizeof(SplitScales) + 255) & ~(size_t)255;

// The exponent for a tensor from its partial maxima; called by all 256 threads of a block.
__device__ __forceinline__ int split_exponent(const uint32_t* partial) {
  __shared__ uint32_t wave_max[4];
  const int tid = threadIdx.x;
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < kAbsMaxBlocks / 256; ++i) m = max(m, partial[tid + 256 * i]);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
  if ((tid & 63) == 0) wave_max[tid >> 6] = m;
  __syncthreads();
  m = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
  // (a denormal largest element counts as 2^-126; an all-zero tensor needs no scale)
  return m == 0 ? 0 : 14 - (max((int)(m >> 23), 1) - 127);
}

// The two terms of v * 2^exponent as f16 bits: hi in the low half of the result, lo in the high half.
__device__ __forceinline__ uint32_t split_f16(float v, int exponent) {
  const float t = ldexpf(v, exponent);
  const _Float16 hi = (_Float16)t;
  const float rest = (t - (float)hi) * 2048.f;
  const _Float16 lo = (_Float16)(fabsf(t) < __builtin_inff() ? rest : 0.f);
  return (uint32_t)__builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
}
// The joined sum, still scaled.
__device__ __forceinline__ float join_f16(float hi, float lo) {
  return fabsf(hi) < __builtin_inff() ? fmaf(lo, 1.f / 2048.f, hi) : hi;
}
// Eight split elements as one 16-byte word per term.
__device__ __forceinline__ void pack_terms(const uint32_t (&v)[8], uint4* hi, uint4* lo) {
  *hi = make_uint4((v[0] & 0xffffu) | v[1] << 16, (v[2] & 0xffffu) | v[3] << 16, (v[4] & 0xffffu) | v[5] << 16,
                   (v[6] & 0xffffu) | v[7] << 16);
  *lo = make_uint4(v[0] >> 16 | (v[1] & 0xffff0000u), v[2] >> 16 | (v[3] & 0xffff0000u), v[4] >> 16 | (v[5] & 0xffff0000u),
                   v[6] >> 16 | (v[7] & 0xffff0000u));
}

}  // namespace vcnn
