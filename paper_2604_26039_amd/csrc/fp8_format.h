// Number formats of the FP8 variant: E8M0 block scales and E4M3 codes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ramp_internal.h"

namespace ramp {

constexpr int kGroup = 128;  // k-values per scale block

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

// Four fp32 -> E4M3 codes in one 32-bit word: round to nearest, ties to even, saturate at 448 (NaN too).  v_cvt_pk_fp8_f32
// rounds that way, but turns values past 448 into NaN, so they are saturated first.
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

typedef int intx8 __attribute__((ext_vector_type(8)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));
typedef short shortx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Largest magnitude bits of two bf16 in a word, kept per half.
__device__ __forceinline__ ushortx2 max_bf16_bits(ushortx2 m, uint32_t two)
{
    return __builtin_elementwise_max(m, __builtin_bit_cast(ushortx2, two & 0x7fff7fffu));
}

// Quantises the 2 * NW values of this lane; its group of 128 lies in the lanes that differ in the bits D0 ... DEND/2 of the lane
// index.  Codes in order, one scale byte, the same bits as e8m0_of_amax and e4m3x4_of_f32 give.  v_cvt_scalef32_pk_fp8_bf16
// divides two bf16 by a power of two and converts them; for finite groups nothing exceeds 448 after that and the codes are the
// same (tests/test_gpu_fp8.py: every bf16 value, scale bytes of the whole range), at a third of the instructions of unpacking,
// scaling and saturating.
// A group with an infinity or NaN takes the general conversion: NaN counts as no magnitude and converts to +-448.
template <int NW, int D0, int DEND>
__device__ __forceinline__ uint32_t quantise_group(const uint32_t *w, uint32_t *codes)
{
    ushortx2 m = {0, 0};
#pragma unroll
    for (int i = 0; i < NW; ++i) m = max_bf16_bits(m, w[i]);
    auto group_max = [](uint32_t v) __attribute__((always_inline)) {
#pragma unroll
        for (int d = D0; d < DEND; d <<= 1) v = max(v, (uint32_t)__shfl_xor((int)v, d));
        return v;
    };
    uint32_t top = group_max(m[0] > m[1] ? m[0] : m[1]);
    if (__builtin_expect(top >= 0x7f80u, 0)) {
        top = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const uint32_t lo = w[i] & 0x7fffu, hi = (w[i] >> 16) & 0x7fffu;
            top = max(top, max(lo > 0x7f80u ? 0u : lo, hi > 0x7f80u ? 0u : hi));
        }
        const uint32_t b = e8m0_of_amax(bf16_bits_to_f32(group_max(top)));
        const float inv = inv_scale_of(b);
#pragma unroll
        for (int i = 0; i < NW / 2; ++i) {
            const float v[4] = {bf16_bits_to_f32(w[2 * i] & 0xffffu) * inv, bf16_bits_to_f32(w[2 * i] >> 16) * inv,
                                bf16_bits_to_f32(w[2 * i + 1] & 0xffffu) * inv, bf16_bits_to_f32(w[2 * i + 1] >> 16) * inv};
            codes[i] = e4m3x4_of_f32(v);
        }
        return b;
    }
    const uint32_t b = e8m0_of_amax(bf16_bits_to_f32(top));
    const float scale = __builtin_bit_cast(float, b << 23);
#pragma unroll
    for (int i = 0; i < NW / 2; ++i) {
        shortx2 r = {0, 0};
        r = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, __builtin_bit_cast(bf16x2, w[2 * i]), scale, false);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, __builtin_bit_cast(bf16x2, w[2 * i + 1]), scale, true);
        codes[i] = __builtin_bit_cast(uint32_t, r);
    }
    return b;
}

// src bf16 [rows, K] row-major -> codes [rows, K], scale bytes [rows, stride].  Bound by memory, and at small sizes by the
// launch: K is a multiple of the group, so the groups are consecutive in both arrays; 16 lanes take one, a 16-byte load and an
// 8-byte store each, and the maximum is four lane exchanges.  The vector types carry the alignment of one value: the
// quantising entry point takes any address.
// first, step: group of the workgroup's first 16 lanes, and groups of the whole launch.
typedef uint32_t UnalignedWords2 __attribute__((ext_vector_type(2), aligned(1)));
__device__ __forceinline__ void quantise_rows(const QuantRows &q, size_t first, size_t step)
{
    const int sub = threadIdx.x & 15;
    const int groups = q.K / kGroup;
    const size_t total = (size_t)q.rows * groups;
    for (size_t g = first + (threadIdx.x >> 4); g < total; g += step) {
        const UnalignedWords4 v = *reinterpret_cast<const UnalignedWords4 *>(q.src + g * kGroup + sub * 8);
        const uint32_t w[4] = {v[0], v[1], v[2], v[3]};
        uint32_t c[2];
        const uint32_t b = quantise_group<4, 1, 16>(w, c);
        *reinterpret_cast<UnalignedWords2 *>(q.codes + g * kGroup + sub * 8) = UnalignedWords2{c[0], c[1]};
        if (sub == 0) {
            const size_t row = (total >> 32) ? g / groups : (uint32_t)g / (uint32_t)groups;
            q.sb[row * (size_t)q.stride + (g - row * groups)] = (uint8_t)b;
        }
    }
}

}  // namespace ramp
