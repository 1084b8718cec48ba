// Number formats of the FP8 variant: E8M0 block scales and E4M3 codes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ramp {

// E8M0 byte of the smallest power of two s with amax / s <= 448 (448 = 1.75 * 2^8): from the fp32 bits of amax.
__device__ __forceinline__ uint32_t e8m0_of_amax(float amax)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, amax) & 0x7fffffffu;
    if (u == 0u || u >= 0x7f800000u) return 127u;  // all-zero block (or not finite): scale 1
    const int field = (int)(u >> 23);
    const int b = field - ((u & 0x7fffffu) <= 0x600000u ? 8 : 7);
    return (uint32_t)(b < 0 ? 0 : (b > 254 ? 254 : b));
}
// 2^(127-b): the factor that brings a block into the E4M3 range.
__device__ __forceinline__ float inv_scale_of(uint32_t b) { return __builtin_bit_cast(float, (254u - b) << 23); }

// fp32 -> E4M3 code: round to nearest, ties to even, saturate at 448.
__device__ __forceinline__ uint32_t e4m3_of_f32(float v)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const uint32_t sign = (u >> 24) & 0x80u;
    uint32_t a = u & 0x7fffffffu;
    if (a > 0x43e00000u) a = 0x43e00000u;  // 448
    if (a >= 0x3c800000u) {                // >= 2^-6: normal code; keep 3 mantissa bits
        const uint32_t r = a + 0x7ffffu + ((a >> 20) & 1u);
        uint32_t code = (r >> 20) - (120u << 3);
        if (code > 0x7eu) code = 0x7eu;
        return sign | code;
    }
    // subnormal range: multiples of 2^-9 (8 of them reach the smallest normal value, code 8)
    const float f = __builtin_bit_cast(float, a) * 512.0f;
    return sign | (uint32_t)__builtin_rintf(f);
}

// Four of them, in one 32-bit word, by the conversion instruction of the chip (v_cvt_pk_fp8_f32): the same rounding, ties
// included; it turns values past 448 into NaN, so they are saturated first.
__device__ __forceinline__ uint32_t e4m3x4_of_f32(const float *v)
{
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t u = __builtin_bit_cast(uint32_t, v[i]);
        const uint32_t a = u & 0x7fffffffu;
        s[i] = __builtin_bit_cast(float, (a > 0x43e00000u ? 0x43e00000u : a) | (u & 0x80000000u));
    }
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(s[0], s[1], 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(s[2], s[3], w, true);
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __builtin_bit_cast(float, h << 16); }

}  // namespace ramp
