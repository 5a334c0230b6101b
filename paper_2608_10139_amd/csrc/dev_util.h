// Device-side helpers shared by the HIP kernel files: 16-bit float bit-pattern
// conversions (round to nearest even) for bf16 and fp16 activations.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aiq {

// activation element types
enum Act : int { ACT_F32 = 0, ACT_BF16 = 1, ACT_F16 = 2 };

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }
__device__ __forceinline__ uint16_t f2h(float f) { return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f)); }
__device__ __forceinline__ float h2f(uint16_t h) { return static_cast<float>(__builtin_bit_cast(_Float16, h)); }

// 16-bit activation of type `act` (ACT_BF16 or ACT_F16)
__device__ __forceinline__ uint16_t f2act(float f, int act) { return act == ACT_F16 ? f2h(f) : f2bf(f); }
__device__ __forceinline__ float act2f(uint16_t v, int act) { return act == ACT_F16 ? h2f(v) : bf2f(v); }

// Lane exchange through a DPP move (a VALU op; a lane shuffle goes through
// the LDS crossbar): 0xB1 lane ^ 1, 0x4E lane ^ 2, 0x141 the mirrored quad of
// eight lanes.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}

// RMSNorm scale of a row from its n_part sums of squares (n_part % 4 == 0,
// 16-byte aligned), added in order.
__device__ __forceinline__ float row_scale(const float* p, int n_part, int d, float eps) {
  float ss = 0.f;
#pragma unroll 4
  for (int k = 0; k < n_part; k += 4) {
    const float4 v = *reinterpret_cast<const float4*>(p + k);
    ss += v.x;
    ss += v.y;
    ss += v.z;
    ss += v.w;
  }
  return 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
}

}  // namespace aiq
