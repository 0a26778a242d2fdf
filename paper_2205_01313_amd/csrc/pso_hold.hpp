// pso_hold.hpp -- runs of a synchronous swarm too large for the resident gang,
// part of whose state stays in registers and LDS (pso_hold.hip).
#pragma once

#include "pso_f64.hpp"
#include "pso_gang.hpp"

namespace pso {

struct HoldShape {
    const void *fn;
    uint32_t G;       // parts: one workgroup per compute unit
    uint32_t slots;   // 16-byte groups of particles per lane
    uint32_t groups;  // of a part
    uint32_t lds_pairs; // dimension pairs of a lane's first group held in LDS
    size_t lds;
};

// Whether a run of T iterations of the swarm beats the grid step this way, and
// its shape (D at most GANG64_MAX_D_ALL).  PSO_HOLD=0 in the environment: never;
// any other value: whatever the size and T.
bool hold_shape(int fitness, const SwarmArgs &a, int64_t T, HoldShape *out);
bool hold_shape(int fitness, const Swarm64Args &a, int64_t T, HoldShape *out);
// 64-bit device words of the meeting.
size_t hold_words(int D);
// Up to T iterations, continuing from and updating the control block, under
// launch_gang's conditions (the parameters within gang_accepts or
// gang64_accepts).
hipError_t launch_hold(const SwarmArgs &a, const HoldShape &s, uint32_t T, unsigned long long *words, hipStream_t stream);
hipError_t launch_hold(const Swarm64Args &a, const HoldShape &s, uint32_t T, hipStream_t stream);

} // namespace pso
