// bf16 <-> fp32 of the element-wise kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace purine {
namespace {
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f2bf(float v) {   // to nearest even; every NaN becomes 0x7FC0
    uint32_t u = __float_as_uint(v);
    uint32_t r = u + 0x7FFFu + ((u >> 16) & 1u);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) r = 0x7FC00000u;
    return (uint16_t)(r >> 16);
}
}  // namespace
}  // namespace purine
