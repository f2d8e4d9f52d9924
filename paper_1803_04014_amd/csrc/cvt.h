// cvt.h -- element conversions FP32 -> FP16 / BF16 bit patterns and back,
// shared by the conversion passes and the GEMMs that split their FP32
// operands while staging them, so both write the same bits.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"

namespace mfg {

__device__ __forceinline__ uint16_t f32_to_f16_bits(float x) {
    return __builtin_bit_cast(uint16_t, (_Float16)x);  // v_cvt_f16_f32, RNE
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float x) {
    uint32_t u = __builtin_bit_cast(uint32_t, x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x0040u);  // quiet NaN
    u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float f16_bits_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

// Four FP32 values -> four 16-bit heads and, with SPLIT, four residuals,
// as the split (and rounding) passes compute each finite element: head =
// RNE(x), residual = RNE((x - head) * 2^11) for FP16, RNE(x - head) for
// BF16, the difference exact in FP32.  Pairs go through gfx950's packed
// conversions (v_cvt_pk_f16_f32 / v_cvt_pk_bf16_f32, round to nearest even),
// which write the MFMA operand's packed layout directly.  (A NaN input gives
// a NaN head whose payload may differ from the passes' sign-keeping quiet
// NaN; every product with it is NaN either way.)
template <bool BF, bool SPLIT>
__device__ __forceinline__ void split4(const f32x4& v, u32x2& h, u32x2& r) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    uint32_t hw[2], rw[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const f2 x = {v[2 * j], v[2 * j + 1]};
        if constexpr (BF) {
            const b2 hh = __builtin_convertvector(x, b2);
            hw[j] = __builtin_bit_cast(uint32_t, hh);
            if constexpr (SPLIT) rw[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x - __builtin_convertvector(hh, f2), b2));
        } else {
            const h2 hh = __builtin_convertvector(x, h2);
            hw[j] = __builtin_bit_cast(uint32_t, hh);
            if constexpr (SPLIT)
                rw[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector((x - __builtin_convertvector(hh, f2)) * 2048.0f, h2));
        }
        if constexpr (!SPLIT) rw[j] = 0u;
    }
    h = u32x2{hw[0], hw[1]};
    r = u32x2{rw[0], rw[1]};
}

}  // namespace mfg
