// A 128 x 128 tile of a product whose operands lie in fragment order, on the half-precision matrix cores.
//
// Fragment order: frag[32-row tile][step of 16 contraction elements][lane][8], word `lane` holding row lane % 32 and
// elements 8 (lane / 32) + 0..7 of the step - what the lane feeds to one MFMA -, one plane per term: TERMS = 2 for
// floats as two f16 terms (split_f16.h; three products per step, the mixed ones in accumulators of their own), 1 for
// bfloat16.  A fragment is 1 KB that goes to LDS by direct loads, a slab ahead, and is read back without bank conflicts.
// Four waves of 64 x 64.  Two slabs of both operands take 64 KB of LDS (two terms: two blocks per CU) or 32 KB (bfloat16,
// one accumulator set: four blocks per CU; with slabs twice as deep and two blocks 16 38 64 64 -> 512 16 16 took 0.74 instead
// of 0.68 ms).
#pragma once
#include "bf16_core.h"
#include "mma_core.h"
#include "split_f16.h"

namespace vcnn {

static constexpr int kFragTile = 128;  // rows and columns of a block's tile: four row tiles of either operand

template <int TERMS>
struct FragSlab {
  static constexpr int STEPS = 2;
  static constexpr int WORDS = 4 * TERMS * STEPS * 64;  // 16-byte words of one operand's slab: four row tiles
  static constexpr size_t LDS_BYTES = 2 * 2 * (size_t)WORDS * 16;
};

// acc = the tile's sums over `slabs` slabs (two terms: still scaled by both operands' powers of two).  fetch_a(sl) /
// fetch_b(sl): the first fragment (term 0) of slab sl in this WAVE's row tile of either operand, plus the lane; steps
// are 64 words apart, terms a_term / b_term.  Ends with every wave past its last read of `lds`.
template <int TERMS, typename FA, typename FB>
__device__ __forceinline__ void frag_product(int slabs, uint4* lds, int64_t a_term, int64_t b_term, FA fetch_a, FB fetch_b,
                                             f32x16 (&acc)[2][2]) {
  constexpr int TM = 2, TN = 2, STEPS = FragSlab<TERMS>::STEPS, WORDS = FragSlab<TERMS>::WORDS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // wave w stages row tile w of both operands: TERMS * STEPS fragments each, 1 KB a load
  auto stage = [&](int sl, uint4* buf) {
    uint4* const to_a = buf + wave * (TERMS * STEPS * 64);
    uint4* const to_b = to_a + WORDS;
    const uint4* const a = fetch_a(sl);
    const uint4* const b = fetch_b(sl);
#pragma unroll
    for (int t = 0; t < TERMS; ++t)
#pragma unroll
      for (int i = 0; i < STEPS; ++i) {
        load_to_lds16(a + t * a_term + i * 64, to_a + (t * STEPS + i) * 64);
        load_to_lds16(b + t * b_term + i * 64, to_b + (t * STEPS + i) * 64);
      }
  };
  f32x16 mixed[TERMS == 2 ? TM : 1][TERMS == 2 ? TN : 1];
  zero_acc<TM, TN>(acc);
  if constexpr (TERMS == 2) zero_acc<TM, TN>(mixed);
  const int ra = (wave & 1) * 2, rb = (wave >> 1) * 2;  // this wave's first row tile of either operand
  stage(0, lds);
  for (int sl = 0; sl < slabs; ++sl) {
    const uint4* const A = lds + (sl & 1) * 2 * WORDS + lane;
    const uint4* const B = A + WORDS;
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share of the slab has landed
    __syncthreads();                     // everyone's has, and the other buffer is free
    if (sl + 1 < slabs) stage(sl + 1, lds + ((sl + 1) & 1) * 2 * WORDS);
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
      uint4 fa[TERMS][TM], fb[TERMS][TN];
#pragma unroll
      for (int t = 0; t < TERMS; ++t) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) fa[t][mi] = A[(((ra + mi) * TERMS + t) * STEPS + i) * 64];
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) fb[t][ni] = B[(((rb + ni) * TERMS + t) * STEPS + i) * 64];
      }
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
          if constexpr (TERMS == 2) {
            acc[mi][ni] = mfma_f16(fa[0][mi], fb[0][ni], acc[mi][ni]);
            mixed[mi][ni] = mfma_f16(fa[0][mi], fb[1][ni], mixed[mi][ni]);
          } else {
            acc[mi][ni] = mfma_bf16(fa[0][mi], fb[0][ni], acc[mi][ni]);
          }
        }
      if constexpr (TERMS == 2) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
          for (int ni = 0; ni < TN; ++ni) mixed[mi][ni] = mfma_f16(fa[1][mi], fb[0][ni], mixed[mi][ni]);
      }
    }
  }
  if constexpr (TERMS == 2) {
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int ni = 0; ni < TN; ++ni)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[mi][ni][q] = join_f16(acc[mi][ni][q], mixed[mi][ni][q]);
  }
  __syncthreads();
}

}  // namespace vcnn
