// pso_launch_length.hpp -- how many iterations of a run one launch of a resident
// gang or of a held run takes (host arithmetic only).
#pragma once

#include <algorithm>
#include <cstdint>

namespace pso {

constexpr uint32_t GANG_PARTS_MAX = 256;  // one byte of the meeting's minimum
constexpr uint32_t GANG_MAX_T = 1u << 23; // meetings are numbered in 24 bits

// Lengths of a run's launches.  Other work on the device waits for the end of a
// launch that has most compute units, so one of more than half of them is kept
// to about MOST_LAUNCH_US, others, which share a hardware queue with other streams
// at most, to about FEW_LAUNCH_US: the first launch of a run by an estimate of an
// iteration's time (gang_iteration_us), the following ones by what the last one
// took, from its launch to its results.  Beside a run of Rastrigin D = 30,
// N = 262144, 200 iterations of Sphere D = 2, N = 300 took, at the median, 49.4 ms
// with launches of 50 ms, 10.0 with 10, 5.6 with 5 and 2.0 with 2 (0.2 alone, and
// beside step launches); a launch more costs 30 to 65 us (its state out and in, the host
// between): 1000 iterations of Rastrigin D = 32, N = 2^20 take 85.7 ms with
// launches of 50 ms, 86.2 with 10, 87.0 with 5 and 89.1 with 2.
constexpr double MOST_LAUNCH_US = 10000.0, FEW_LAUNCH_US = 20000.0;
struct LaunchLength {
    double launch_us, iteration_us;
    // of a run of `left` more iterations; a remainder of a quarter is taken along
    int64_t next(int64_t left) const
    {
        const int64_t T = std::max<int64_t>(1, (int64_t)std::min(launch_us / iteration_us, 0.8 * GANG_MAX_T));
        return left <= T + T / 4 ? left : T;
    }
    // the first also waited for what the stream held before it, so the time
    // falls back by at most a factor of four a launch
    void took(int64_t T, double us) { iteration_us = std::max(us / (double)T, 0.25 * iteration_us); }
};
// The launch time of a gang or held run of so many parts.
inline double launch_us(uint32_t parts) { return parts > GANG_PARTS_MAX / 2 ? MOST_LAUNCH_US : FEW_LAUNCH_US; }
// An upper estimate of an iteration's time.  The slowest function measured, us
// per iteration of the first hundred, and the estimate: binary32 N = 1024, D = 2
// 2.0 / 1.6; 1000 x 30 4.5 / 4.5; 1000 x 128 7.1 / 9.6; 32768 x 128 11.6 / 14.9;
// 65536 x 128 17.4 / 20.3; 262144 x 30 14.0 / 14.7; held 2^20 x 4 28 / 22, x 32 94 /
// 117; binary64 200 x 30 5.5 / 5.8; 1000 x 128 10.5 / 12.7; 32768 x 128 26 / 45;
// 262144 x 30 44 / 69; held 2^20 x 32 238 / 274.
inline double gang_iteration_us(double N, int D, bool held, bool wide)
{
    const double m = N * D * 1e-6;
    if (wide) return (D > 2 ? 4.0 : 2.0) + 0.06 * D + 8.0 * m;
    return held ? 8.0 + 0.05 * D + 3.2 * m : (D > 2 ? 3.0 : 1.5) + 0.05 * D + 1.3 * m;
}

} // namespace pso
