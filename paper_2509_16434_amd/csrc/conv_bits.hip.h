// Device helpers shared by the convolution kernels: clamping and rounding, mask bits, the permutation of LDS pixels.
#pragma once
#include "common.hip.h"
#include "gemm_dma.hip.h"

// bf16 pair of (max(lo, 0), max(hi, 0)): rounded first, then clamped as 16-bit integers (a negative bf16 is a
// negative int16, and rounding keeps the sign, so the order of rounding and clamping does not matter)
__device__ __forceinline__ uint32_t relu_pack2bf(float lo, float hi) {
  typedef short s16x2_t __attribute__((ext_vector_type(2)));
  const s16x2_t z = {0, 0};
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2_t, pack2bf(lo, hi)), z));
}
// Which of the four non-negative bf16 of the pairs (x, y) are non-zero, as bits 0..3 times the weight the caller's
// negw encodes (nonzero_weights: 1, or 16 for the upper nibble of a byte), added to acc.  A half is at most 0x7fff, so
// x + 0x7fff7fff carries "non-zero" into each half's top bit without a carry between the halves; the byte permute's
// sign selectors spread the four top bits to bytes 0x00 / 0xff (= -1), and the signed 4-byte dot product with the
// weights -1, -2, -4, -8 (or -16 .. -128) sums them.
// x of this lane OR x of the lane 32 away (one half-wave swap instead of a permute through LDS): either returned half
// holds the own value and the other the partner's, so the OR of both is independent of which is which
__device__ __forceinline__ uint32_t or_with_lane_xor32(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return r[0] | r[1];
}
__device__ __forceinline__ uint32_t nonzero_weights(int upper) { return upper ? 0x80c0e0f0u : 0xf8fcfeffu; }
__device__ __forceinline__ uint32_t nonzero_signs(uint32_t x, uint32_t y) { return __builtin_amdgcn_perm(y + 0x7fff7fffu, x + 0x7fff7fffu, 0x0b0a0908u); }
__device__ __forceinline__ uint32_t nonzero4(uint32_t x, uint32_t y, uint32_t negw) {
  return (uint32_t)__builtin_amdgcn_sdot4((int)nonzero_signs(x, y), (int)negw, 0, false);
}

// LDS image rows hold pixel slots of CIN*2 bytes (slot 0 and slot W+1 are zero pads).  A byte at
// logical in-row offset `off` is stored at off ^ tile_swz_bits<CIN>(off): the 16-byte chunks of a
// pixel are permuted by bits of the slot index (which the permutation leaves unchanged, so it is
// its own inverse).  Reads that walk over every second slot then use all banks evenly, two lanes
// per bank group.
template <int CIN>
__device__ __forceinline__ uint32_t tile_swz_bits(uint32_t off) {
  if (CIN == 32) return ((off >> 8) & 3u) << 4;          // slot >> 2
  const uint32_t t = (off >> 8) & 7u;                    // slot >> 1
  return (((t & 1u) << 2) | (t >> 1)) << 4;              // rotated, so neighbours differ in the top bit
}
