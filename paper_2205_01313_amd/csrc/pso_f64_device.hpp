// pso_f64_device.hpp -- device building blocks of the binary64 path: order
// bits, cos(pi y), the fitness functions and lexicographic minima of (order
// bits, particle index).
#pragma once

#include <cmath>

#include "pso_device.hpp"

namespace pso {

constexpr uint32_t NO_IDX = 0xFFFFFFFFu;

// Order bits of a binary64: unsigned order = numeric order, -0 = +0, NaN last.
__device__ __forceinline__ unsigned long long ord64(double f)
{
    if (f != f) return ~0ull;
    if (f == 0.0) f = 0.0;
    const unsigned long long b = (unsigned long long)__double_as_longlong(f);
    return (b & 0x8000000000000000ull) ? ~b : (b | 0x8000000000000000ull);
}

// Inverse of ord64 (for non-NaN values; -0 comes back as +0).
__device__ __forceinline__ double ord64_value(unsigned long long o)
{
    const unsigned long long b = (o & 0x8000000000000000ull) ? (o & 0x7FFFFFFFFFFFFFFFull) : ~o;
    return __longlong_as_double((long long)b);
}

__device__ __forceinline__ double clampd(double v, double lo, double hi)
{
    v = (v < lo) ? lo : v;
    return (v > hi) ? hi : v;
}

// cos(pi y) after the exact reduction y = n + r.
__device__ __forceinline__ double cospi64(double y)
{
    const double n = rint(y);
    const double r = y - n;
    const double c = cos(M_PI * r);
    const double h = 0.5 * n; // an integer iff n is even
    return h - rint(h) != 0.0 ? -c : c;
}

// The fitness functions in binary64, accumulated in dimension order.
template <int FIT>
struct Fitness64 {
    double acc = 0.0, aux = 0.0;

    __device__ __forceinline__ void add(double z, int d)
    {
        if constexpr (FIT == F_SPHERE) {
            acc = acc + z * z;
        } else if constexpr (FIT == F_RASTRIGIN) {
            acc = acc + (z * z - 10.0 * cospi64(2.0 * z));
        } else if constexpr (FIT == F_ROSENBROCK) {
            if (d > 0) {
                const double a = z - aux * aux;
                const double b = 1.0 - aux;
                acc = acc + (100.0 * a * a + b * b);
            }
            aux = z;
        } else if constexpr (FIT == F_ACKLEY) {
            acc = acc + z * z;
            aux = aux + cospi64(2.0 * z);
        } else {
            acc = acc + (z * z * z - 0.8 * z * z - 1000.0 * z + 8000.0);
        }
    }

    __device__ __forceinline__ double value(int D) const
    {
        if constexpr (FIT == F_RASTRIGIN) {
            return 10.0 * D + acc;
        } else if constexpr (FIT == F_ACKLEY) {
            return 20.0 - 20.0 * exp(-0.2 * sqrt(acc / D)) + M_E - exp(aux / D);
        } else if constexpr (FIT == F_CUBIC) {
            return -acc; // Eq. 3, negated: the paper maximises it
        } else {
            return acc;
        }
    }
};

__device__ __forceinline__ void lexmin(unsigned long long &k, uint32_t &i, unsigned long long k2, uint32_t i2)
{
    if (k2 < k || (k2 == k && i2 < i)) {
        k = k2;
        i = i2;
    }
}

// Wavefront lexicographic minimum of the candidates (lanes with i != NO_IDX,
// k != ~0) in every lane.  Beating the gbest is rare after the first
// iterations, so a wavefront with no candidate or one takes no shuffles.
__device__ __forceinline__ void wave_lexmin_sparse(unsigned long long &k, uint32_t &i)
{
    const unsigned long long m = __ballot(i != NO_IDX);
    if (m == 0) {
        k = ~0ull;
        i = NO_IDX;
    } else if ((m & (m - 1)) == 0) {
        const int l = __builtin_ctzll(m);
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)k, l), hi = __builtin_amdgcn_readlane((uint32_t)(k >> 32), l);
        k = ((unsigned long long)hi << 32) | lo;
        i = __builtin_amdgcn_readlane(i, l);
    } else {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const unsigned long long k2 = __shfl_xor(k, off, 64);
            const uint32_t i2 = __shfl_xor(i, off, 64);
            lexmin(k, i, k2, i2);
        }
    }
}

} // namespace pso
