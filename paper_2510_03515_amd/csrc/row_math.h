// Rows of bf16 values in 16-byte chunks: unpacking, rounding, packing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rapid {

__device__ inline void unpack8(const uint4& v, float (&f)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = __builtin_bit_cast(float, w[e] << 16);
        f[2 * e + 1] = __builtin_bit_cast(float, w[e] & 0xffff0000u);
    }
}

// double -> float such that rounding the float to bf16 (nearest even) gives what rounding the double to bf16 directly
// would.  The float nearest to v lies on the same side of every midpoint of two bf16 values as v does, or on it: there, and if
// v itself is not the midpoint, it is moved off towards v (about one element in 65536).
__device__ inline float round_for_bf16(double v) {
    const float f = (float)v;
    const uint32_t b = __builtin_bit_cast(uint32_t, f);
    if ((b & 0xffffu) != 0x8000u || (double)f == v || !isfinite(f)) return f;
    return __builtin_bit_cast(float, fabs((double)f) > fabs(v) ? b - 1u : b + 1u);
}

__device__ inline uint32_t pack2(float a, float b) {
    const __bf16 x = (__bf16)a, y = (__bf16)b;
    return (uint32_t)__builtin_bit_cast(unsigned short, x) | ((uint32_t)__builtin_bit_cast(unsigned short, y) << 16);
}

__device__ inline uint4 pack8(const float (&f)[8]) {
    return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
}

}  // namespace rapid
