// What the fp32 kernels share: the matrix instruction, its operand layout (see s2attn_f32.hip) and the
// loads and stores of a wave's own 16 rows.
#pragma once
#include "s2attn_bf16_common.h"
#include "s2attn_device.h"

namespace s2 {

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Sum / maximum over the four lanes that share a column (lanes c16 + 16 q4).
__device__ __forceinline__ float sum_cols(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}
__device__ __forceinline__ float max_cols(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}

// The wave's own 16 rows as B operand: X[row][16 i + 4 q4 ..] straight from global memory.
template <int D>
__device__ __forceinline__ void load_own(f32x4 (&own)[D / 16], const void* src, size_t off, int q4) {
  const float* p = static_cast<const float*>(src) + off + 4 * q4;
#pragma unroll
  for (int i = 0; i < D / 16; ++i) own[i] = *reinterpret_cast<const f32x4*>(p + 16 * i);
}

// Stores the accumulators of the lane's row (column c16 of C): 16 consecutive d per j.
template <int D>
__device__ __forceinline__ void store_row(float* dst, const f32x4 (&acc)[D / 64][4], float mul, int q4) {
#pragma unroll
  for (int j = 0; j < D / 64; ++j)
#pragma unroll
    for (int w = 0; w < 4; ++w)
      *reinterpret_cast<float4*>(dst + 64 * j + 16 * q4 + 4 * w) =
          make_float4(acc[j][0][w] * mul, acc[j][1][w] * mul, acc[j][2][w] * mul, acc[j][3][w] * mul);
}

}  // namespace s2
