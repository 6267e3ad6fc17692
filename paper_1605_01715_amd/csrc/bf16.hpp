// bfloat16 parts of float32 values (split-BF16 M2L), device code.
#pragma once

#include "common.hpp"

namespace fmm {

// float32 -> bfloat16, round to nearest even (finite inputs)
__device__ inline uint16_t f2bf(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// x = h + m + l up to 2^-24 |x| (each residual is exact in float32); the
// two-part split is h and m (x = h + m up to 2^-16 |x|)
__device__ inline void split3(float x, uint16_t &h, uint16_t &m, uint16_t &l) {
    h = f2bf(x);
    float r1 = x - bf2f(h);
    m = f2bf(r1);
    l = f2bf(r1 - bf2f(m));
}

// Split-BF16 vector layout: per vector of r_pad values, per 32 values, NP parts
// of 32 bfloat16 (64 NP bytes). vec_bf_stride: elements per vector.
__host__ __device__ constexpr int64_t vec_bf_stride(int r_pad, int np) { return np * (int64_t)r_pad; }

}  // namespace fmm
