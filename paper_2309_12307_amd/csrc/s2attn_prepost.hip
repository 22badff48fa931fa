// Backward pre-pass of the bf16 path and post-pass of both paths.
//   delta:   the row term of the softmax Jacobian, delta_i = sum_j P_ij dP_ij = dO_i . O_i;
//            stored negated, as the dP accumulators of dK/dV start with it; the same pass
//            rescales lse to base 2 for the kernels' exp2
//   combine: sum of the fp32 partials of dK/dV when the query heads of a kv head are cut into
//            parts (always when one kv head serves both shifted and unshifted query heads).
// Both are pure streaming kernels (HBM-bound, 16-byte coalesced accesses).
#include "s2attn_device.h"
#include "s2attn_launch.h"
#include "s2attn.h"

namespace s2 {
namespace {

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t hi16) { return __uint_as_float(hi16 << 16); }

__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {   // round to nearest even
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// A workgroup takes kRows / HEADS consecutive tokens of HEADS neighbouring heads, D / 8 lanes to a row, so
// that the row terms (and lse) are whole lines and the rows it reads pairs of neighbours in memory;
// neighbouring workgroups take the other heads of the same tokens.  Every lane has its eight loads out
// before it waits.  Two heads rather than one or four: D = 128, H = 32, N = 32768 112 us, 121 and 117
// (one row per 16 lanes, sixteen heads to a workgroup: 111); N = 4096, B = 2 23.6, 24.9 and 23.7 (28.5).
template <int D, int HEADS>
__global__ void __launch_bounds__(256) delta_kernel(const void* o, const void* dout, const float* lse,
                                                    float* neg_delta, float* lse2, int N, int H, Div by_heads,
                                                    Div by_tiles, int tiles) {
  constexpr int kLanes = D / 8, kPass = 256 / kLanes, kRows = 4 * kPass, kTokens = kRows / HEADS;
  __shared__ float sums[kRows];
  const int tid = thread_id();
  const int bt = quot(block_id(), by_heads), h0 = (block_id() - bt * (H / HEADS)) * HEADS;
  const int b = quot(bt, by_tiles), t0 = (bt - b * tiles) * kTokens;
  const int sub = tid / kLanes, lane = tid % kLanes;
  // row terms of thread tid < kRows: token tid % kTokens of head tid / kTokens
  const bool row = tid < kRows && t0 + tid % kTokens < N;
  const size_t at = ((size_t)b * H + h0 + tid / kTokens) * N + t0 + tid % kTokens;
  uint4 x[4], y[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = p * kPass + sub, h = h0 + r % HEADS;
    const int t = min(t0 + r / HEADS, N - 1);
    const size_t off = (((size_t)b * N + t) * H + h) * D;
    x[p] = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(o) + off)[lane];
    y[p] = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(dout) + off)[lane];
  }
  const float l = row ? lse[at] : 0.f;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const uint32_t xs[4] = {x[p].x, x[p].y, x[p].z, x[p].w}, ys[4] = {y[p].x, y[p].y, y[p].z, y[p].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[p] += bf16_bits_to_f32(xs[e] & 0xFFFFu) * bf16_bits_to_f32(ys[e] & 0xFFFFu);
      acc[p] += bf16_bits_to_f32(xs[e] >> 16) * bf16_bits_to_f32(ys[e] >> 16);
    }
  }
#pragma unroll
  for (int m = 1; m < kLanes; m *= 2)
#pragma unroll
    for (int p = 0; p < 4; ++p) acc[p] += __shfl_xor(acc[p], m);
  if (lane == 0)
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int r = p * kPass + sub;
      sums[r % HEADS * kTokens + r / HEADS] = acc[p];
    }
  __syncthreads();
  if (row) {
    neg_delta[at] = -sums[tid];
    lse2[at] = l * 1.4426950408889634f;
  }
}

// dk (dv) = sum of the `parts` contiguous fp32 partials, in order.
template <bool BF16>
__global__ void __launch_bounds__(256) combine_kernel(const float* partial, void* dk, void* dv, TStride sdk,
                                                      TStride sdv, int N, int Hkv, int D, int parts, size_t elems) {
  const size_t i4 = ((size_t)block_id() * 256 + thread_id()) * 4;
  if (i4 >= elems) return;
  // contiguous (b, t, c, d) index of the partials -> row of the (possibly strided) output
  const int d = (int)(i4 % D);
  const size_t row = i4 / D;
  const int c = (int)(row % Hkv);
  const size_t bt = row / Hkv;
  const int t = (int)(bt % N), b = (int)(bt / N);
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const float* src = partial + (size_t)(which * parts) * elems + i4;
    float4 r = *reinterpret_cast<const float4*>(src);
    for (int p = 1; p < parts; ++p) {
      const float4 x = *reinterpret_cast<const float4*>(src + p * elems);
      r.x += x.x; r.y += x.y; r.z += x.z; r.w += x.w;
    }
    void* out = which == 0 ? dk : dv;
    const size_t o = row_off(which == 0 ? sdk : sdv, b, t, c) + d;
    if (BF16) {
      uint2 pk;
      pk.x = f32_to_bf16_bits(r.x) | (f32_to_bf16_bits(r.y) << 16);
      pk.y = f32_to_bf16_bits(r.z) | (f32_to_bf16_bits(r.w) << 16);
      *reinterpret_cast<uint2*>(static_cast<uint16_t*>(out) + o) = pk;
    } else {
      *reinterpret_cast<float4*>(static_cast<float*>(out) + o) = r;
    }
  }
}

}  // namespace

template <int D, int HEADS>
static int launch_delta_t(const KArgs& a, hipStream_t st) {
  constexpr int tokens = 4 * 256 / (D / 8) / HEADS;
  const int tiles = (a.N + tokens - 1) / tokens;
  hipLaunchKernelGGL((delta_kernel<D, HEADS>), dim3((unsigned)(a.B * tiles * (a.H / HEADS))), dim3(256), 0, st, a.o, a.dout,
                     a.lse, a.neg_delta, a.lse2, a.N, a.H, div_by(a.H / HEADS), div_by(tiles), tiles);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_delta_bf16(const KArgs& a, hipStream_t st) {
  if (a.H % 2 != 0) return a.D == 64 ? launch_delta_t<64, 1>(a, st) : launch_delta_t<128, 1>(a, st);
  return a.D == 64 ? launch_delta_t<64, 2>(a, st) : launch_delta_t<128, 2>(a, st);
}

int launch_combine_partials(const KArgs& a, int dtype, hipStream_t st) {
  const size_t elems = (size_t)a.B * a.N * a.Hkv * a.D;
  dim3 grid((unsigned)((elems / 4 + 255) / 256));
  if (dtype == S2ATTN_BF16)
    hipLaunchKernelGGL(combine_kernel<true>, grid, dim3(256), 0, st, a.dkv_partial, a.dk, a.dv, a.sdk, a.sdv, a.N,
                       a.Hkv, a.D, a.parts, elems);
  else
    hipLaunchKernelGGL(combine_kernel<false>, grid, dim3(256), 0, st, a.dkv_partial, a.dk, a.dv, a.sdk, a.sdv, a.N,
                       a.Hkv, a.D, a.parts, elems);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace s2
