// The layer's 16-bit element types (dtype 1 = fp16, 2 = bf16) to and from fp32.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cc {

template <int DT>
__device__ __forceinline__ float to_f32(uint16_t v)
{
    if constexpr (DT == 1) return float(__builtin_bit_cast(_Float16, v));
    else return __uint_as_float(uint32_t(v) << 16);
}

template <int DT>
__device__ __forceinline__ uint16_t from_f32(float v)
{
    if constexpr (DT == 1) {
        return __builtin_bit_cast(uint16_t, _Float16(v));  // round to nearest even
    } else {
        const uint32_t b = __float_as_uint(v);
        if ((b & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
        return uint16_t((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
    }
}

}  // namespace cc
