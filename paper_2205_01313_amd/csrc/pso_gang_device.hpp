// pso_gang_device.hpp -- the shorter instruction sequences of the kernels that
// hold a swarm in registers, exact where short_forms_exact says so.
#pragma once

#include "pso_device.hpp"

namespace pso {

// cos(2 pi z) for |2 z| < 2^22: cospi_f32's operations without the cases of
// large and non-finite arguments (NaN gives NaN).  2z + 1.5 2^23 rounds 2z to
// an integer and leaves its parity in the lowest bit.
__device__ __forceinline__ float cos2pi_small(float z)
{
    const float t = __builtin_fmaf(z, 2.0f, 0x1.8p23f);
    const float n = t - 0x1.8p23f;
    const float a = __builtin_fabsf(__builtin_fmaf(z, 2.0f, -n));
    const bool lo = a <= 0.25f;
    const float cc = cos_pi_series(a), ss = sin_pi_series(0.5f - a);
    return __uint_as_float(__float_as_uint(lo ? cc : ss) ^ (__float_as_uint(t) << 31));
}

// The fitness term(s) of one dimension, and Rosenbrock's of a pair: the
// expressions Fitness<FIT>::add evaluates.
template <int FIT>
__device__ __forceinline__ float gang_term(float z)
{
    if constexpr (FIT == F_RASTRIGIN) return z * z - 10.0f * cos2pi_small(z);
    else if constexpr (FIT == F_CUBIC) {
        const float z2 = z * z;
        return ((z2 * z - 0.8f * z2) - 1000.0f * z) + 8000.0f;
    } else return z * z; // Sphere, Ackley's first word
}

__device__ __forceinline__ float rosen_term(float z, float zp)
{
    const float a = z - zp * zp;
    const float b = 1.0f - zp;
    return 100.0f * (a * a) + b * b;
}

// Clamp to [lo, hi] in two instructions; equals the comparisons for every
// value the gang accepts (gang_accepts: signs of zero).
__device__ __forceinline__ float clamp_pos(float v, float lo, float hi)
{
    return __builtin_elementwise_minimum(__builtin_elementwise_maximum(v, lo), hi);
}

} // namespace pso
