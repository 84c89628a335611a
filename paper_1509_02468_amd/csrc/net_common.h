// Shared by the network's training pass (net_train.hip) and inference (net.hip):
// the flat weight layout, the MFMA operand types and products, BF16 rounding and
// the index arithmetic of a tile.
#pragma once

#include "gsf_internal.h"

namespace gsf {

// W1[o][c][ky][kx], W2[o][c][ky][kx], W3[c][ky][kx]
constexpr int kOffW1 = 0, kOffW2 = 288, kOffW3 = 2592, kNetWeights = 2736;

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx2_t __attribute__((ext_vector_type(2)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

// two FP32 values rounded to BF16 (nearest even), the first in the low half
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  const floatx2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// ReLU that keeps NaN (a NaN inside the network reaches its output, where it
// triggers the T = I fallback)
__device__ __forceinline__ float relu(float v) { return __builtin_elementwise_maximum(v, 0.0f); }

// 16 x 16 products over K = 32 BF16 values
__device__ __forceinline__ floatx4_t mfma_bf16_k32(uint4_t a, uint4_t b, floatx4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                 0, 0, 0);
}

// i / D for the small pixel indexes of a tile (0 <= i < N): one 24-bit product
// and a shift (a general division by a constant takes a 64-bit product)
constexpr bool div_exact(int d, int n) {
  for (int i = 0; i < n; ++i)
    if (i / d != (i * ((65536 + d - 1) / d)) >> 16) return false;
  return true;
}
template <int D, int N>
__device__ __forceinline__ int div_px(int i) {
  static_assert(div_exact(D, N), "the reciprocal is exact over the range");
  return __mul24(i, (65536 + D - 1) / D) >> 16;
}

}  // namespace gsf
