// What the attention kernels share: maxima and sums over the halves of a wave, the bound of the late rescaling.
#pragma once
#include "gemm_mfma.h"

// The two halves of a wave (lanes l and l + 32) without a trip through LDS.  swap_halves(a, b): first result: a in the lower half and b of the lower
// half in the upper one; second: a of the upper half in the lower one and b in the upper half.
__device__ __forceinline__ u32x2 swap_halves(uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  return u32x2{r[0], r[1]};
#else
  return u32x2{a, b};
#endif
}
__device__ __forceinline__ float max_halves(float v) {
  const u32x2 r = swap_halves(__float_as_uint(v), __float_as_uint(v));
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float v) {
  const u32x2 r = swap_halves(__float_as_uint(v), __float_as_uint(v));
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Online softmax of the attention kernels: accumulators and sums are rescaled only when a row's maximum has risen by more than 2^8 over the one they
// refer to (log2 units), the conditional rescaling of FlashAttention-4.  Probabilities are then up to 256 and not up to 1, sums and accumulators by the same factor: float16 and float32 round
// them just as well, and small ones are further from float16's subnormals.  With the rescaling at every rise (64 multiplications per tile and
// wave), one of 32 rows rose in most tiles of a chunk.
constexpr float kLateRescale = 8.f;
