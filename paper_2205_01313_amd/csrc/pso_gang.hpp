// pso_gang.hpp -- the resident gang: a synchronous swarm's whole pso_run by
// co-resident workgroups that hold it in registers (pso_gang.hip).
#pragma once

#include <algorithm>

#include "pso_kernels.hpp"
#include "pso_launch_length.hpp"

namespace pso {

// Ctrl::gang_state of a gang launch once its parts have met or given up.
constexpr unsigned int GANG_GO = 1u;     // all parts resident: the launch ran
constexpr unsigned int GANG_ABSENT = 2u; // not all resident in time: nothing was touched

constexpr unsigned long long GANG_TICKS = 2000000000ull;   // 20 s of the 100 MHz wall clock: a part is lost
// 0.5 ms: the parts are not resident together.  All of them arrive within 0.05 ms
// on an idle device, also after seconds of rest (but for a kernel's first launch);
// what waits in vain holds compute units that another kernel could use.
constexpr unsigned long long RENDEZVOUS_TICKS = 50000ull;
constexpr int SPEC_MAX_K = 64;                             // iterations of a block at most (fits the word's 8 bits)
constexpr int KEY_STRIDE = 8;                              // key words one per 64-byte line

// Dimensions are taken in groups of four (all of C < 4): a group is skipped
// whole past D, and otherwise computed whole -- two independent Philox draws
// in straight-line code; dimensions of it past D hold values that nothing
// reads.
constexpr int group_of(int C) { return C < 4 ? C : 4; }

// Iterations of the next block, after one that committed nc iterations and
// ended with a change of the gbest or without: sqrt(mean * ratio), the mean
// number of iterations between changes halved towards each new one and never
// below the iterations since the last.  The same in every part.
__device__ __forceinline__ int next_block(bool changed, int nc, float ratio, float &mean, float &since)
{
    since += (float)nc;
    if (changed) {
        mean = 0.5f * (mean + since);
        since = 0.0f;
    } else {
        mean = __builtin_fmaxf(mean, since);
    }
    const int k = (int)__builtin_sqrtf(mean * ratio);
    return k < 1 ? 1 : (k > SPEC_MAX_K ? SPEC_MAX_K : k);
}
// M / I of a shape (weight: an iteration's work against binary32 Sphere's).
float block_ratio(int C, uint32_t L, uint32_t lanes, uint32_t G, float weight);

struct GangArgs {
    uint32_t T;                // iterations of the launch (at most GANG_MAX_T)
    uint32_t P, L;             // particles per part, lanes per particle
    float block_ratio;         // a meeting's time over an iteration's
    float c1s, c2s;            // c1 2^-24, c2 2^-24 (exact)
    unsigned long long *words; // the parts' meeting words
};

// How a swarm is laid out over the parts: chunks of C dimensions, P particles
// and P * L lanes per part (rounded up to whole wavefronts), G parts.
struct GangShape {
    const void *fn;
    int C;
    uint32_t P, L, G, lanes;
    size_t lds;
};

// Whether the gang computes this swarm's bits (parameters and box in the
// ranges its shorter instruction sequences are exact for; shift_max: largest
// magnitude of the shift vector; state_set: pso_set_state was called).
bool gang_accepts(int fitness, const SwarmArgs &a, float shift_max, bool state_set);
// The swarm's shape for a run of T iterations, t0 after Step 1, or false if none
// holds it or other paths are faster.
bool gang_shape(int fitness, const SwarmArgs &a, int64_t t0, int64_t T, GangShape *out);
// 64-bit device words of the meeting.
size_t gang_words(uint32_t parts, int D);
// Sphere and Rosenbrock go down one valley and improve their gbest in most of
// the first 500 to 1000 iterations, where the others settle after 100 to 200.
// Every change is a meeting, so while it lasts fewer parts are better.
inline bool settles_late(int fitness) { return fitness == 0 || fitness == 2; } // PSO_SPHERE, PSO_ROSENBROCK
// A swarm small enough for one part: layout(C, P) with its particles packed
// (whole wavefronts where a lane holds a particle) and the smallest chunk that
// fits, from C = 4 on for D > 12, whose fold is shorter that way.  most2, most4
// and most8: the most particles of one part at D <= 2, at D <= 4 and at C = 8.
template <class F>
inline bool one_part(uint32_t N, int D, uint32_t most2, uint32_t most4, uint32_t most8, F &&layout)
{
    const uint32_t whole = (N + 63) / 64 * 64, packed = std::max(16u, (N + 3) / 4 * 4);
    if (D <= 2) return N <= most2 && layout(D, whole);
    if (D <= 4) return N <= 512 ? layout(2, packed) : N <= most4 && layout(4, whole);
    for (int c = D <= 12 ? 2 : 4; c <= 8; c *= 2) {
        const uint32_t L = ((uint32_t)D + c - 1) / c;
        if (c == 8 && (N > most8 || (uint64_t)N * D > 6500)) return false;
        if (L > 1 && packed * L <= 1024 && layout(c, packed)) return true;
    }
    return false;
}

// Compute units of the current device and the most LDS a workgroup may have.
bool gang_device(int *cus, int *lds);
// Up to T iterations, continuing from and updating the control block (stop
// rule included).  ctrl->gang_arrive and gang_state must be zero (launch_arm,
// launch_gang_arm); gang_state then says whether the launch ran.
hipError_t launch_gang(const SwarmArgs &a, const GangShape &s, uint32_t T, unsigned long long *words,
                       hipStream_t stream);

} // namespace pso
