// pso_gang.hpp -- the resident gang: a synchronous swarm's whole pso_run by
// co-resident workgroups that hold it in registers (pso_gang.hip).
#pragma once

#include "pso_kernels.hpp"

namespace pso {

// Ctrl::gang_state of a gang launch once its parts have met or given up.
constexpr unsigned int GANG_GO = 1u;     // all parts resident: the launch ran
constexpr unsigned int GANG_ABSENT = 2u; // not all resident in time: nothing was touched

struct GangArgs {
    uint32_t T;                // iterations of the launch (at most GANG_MAX_T)
    uint32_t P, L;             // particles per part, lanes per particle
    float c1s, c2s;            // c1 2^-24, c2 2^-24 (exact)
    unsigned long long *words; // the parts' meeting words
};
constexpr uint32_t GANG_MAX_T = 1u << 23; // meetings are numbered in 24 bits

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
// The swarm's shape, or false if none holds it.
bool gang_shape(int fitness, const SwarmArgs &a, GangShape *out);
// 64-bit device words of the meeting.
size_t gang_words(uint32_t parts, int D);
// Up to T iterations, continuing from and updating the control block (stop
// rule included).  ctrl->gang_arrive and gang_state must be zero (launch_arm,
// launch_gang_arm); gang_state then says whether the launch ran.
hipError_t launch_gang(const SwarmArgs &a, const GangShape &s, uint32_t T, unsigned long long *words,
                       hipStream_t stream);

} // namespace pso
