// pso_f64.hpp -- the binary64 path: the same method in double (the paper's
// own precision, Sec. 5), from the same binary32 parameters and the same
// 24-bit uniforms.  Host side of the kernels in pso_f64.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pso {

// Control block of a binary64 swarm (device memory).
struct alignas(256) Ctrl64 {
    unsigned long long gord; // order bits of the gbest fitness (see ord64)
    uint32_t gidx;           // gbest particle
    uint32_t arrive;         // workgroups that finished the current launch
    long long giter;         // iteration of the last gbest change
    long long t;             // iterations completed
    uint32_t stop;           // stop rule met
    uint32_t err;            // a bounded wait of the gang kernel gave up
    double tol, fstar;       // stop rule |gbest - fstar| < tol (tol <= 0: off)
    unsigned long long gang_arrive; // gang kernel: workgroup arrivals (monotonic within a launch)
    uint32_t gang_here, gang_state; // resident gang: parts at a launch's rendezvous, its outcome (GANG_GO, GANG_ABSENT)
    long long run_t0;        // iterations completed when the current run was armed
    unsigned char pad2[168];
};
static_assert(sizeof(Ctrl64) == 256, "Ctrl64 layout");

struct Swarm64Args {
    double *x, *v, *p, *pf;        // D*Np, D*Np, D*Np, Np; element (d, i) at d*Np + i
    double *gpos;                  // D
    const double *shift;           // D
    unsigned long long *slot_ord;  // one per grid workgroup (gang: two per workgroup by parity)
    uint32_t *slot_idx;            // as slot_ord
    double *cand_pos;              // gang: [parity][workgroup][D] candidate positions
    unsigned long long *gang_words; // resident gang: the parts' meeting words (null: none)
    uint8_t *pend;                 // Np: 1 = pbest position of i is x, not yet in p (wide grid step)
    Ctrl64 *ctrl;
    uint32_t N, Np;
    int32_t D;
    double lo, hi, w, c1, c2, vmax;
    uint32_t k0, k1;
};

struct Layout64 {
    size_t ctrl, gpos, shift, slot_ord, slot_idx, cand_pos, gang_words, pf, pend, x, v, p, total;
    uint64_t Np;
    uint32_t nblocks;
};

Layout64 layout64_of(uint64_t N, int D);
Swarm64Args bind64(void *base, const Layout64 &L, uint64_t N, int D);

// Step 1 (grid), one iteration (grid), or up to T iterations in one
// workgroup (block).  All honour and update the control block's stop rule.
hipError_t launch64_reset(const Swarm64Args &a, hipStream_t stream);
hipError_t launch64_init(int fitness, const Swarm64Args &a, hipStream_t stream);
hipError_t launch64_step(int fitness, const Swarm64Args &a, hipStream_t stream);
hipError_t launch64_block_run(int fitness, const Swarm64Args &a, long long T, hipStream_t stream);
// The swarm's state fits the LDS of the one-workgroup run (and staging is on).
bool block64_staged_fits(const Swarm64Args &a);
// The grid step of the swarm is the split one (lanes share a particle).
bool step64_split(int fitness, const Swarm64Args &a);
hipError_t launch64_arm(const Swarm64Args &a, double tol, double fstar, hipStream_t stream);
// Copies every pending pbest position (wide grid step) from x to p and
// clears the marks: before the state is read or another path runs.
hipError_t launch64_flush(const Swarm64Args &a, hipStream_t stream);
// out[m] = F(pts[m]) in binary64 for M device-resident points (row-major M x D).
hipError_t launch64_eval(int fitness, const Swarm64Args &a, const double *pts, uint64_t M, double *out,
                         hipStream_t stream);
// Up to T iterations by a persistent gang of co-resident workgroups that meet
// once per iteration (bit-identical to T grid steps); ctrl->gang_arrive must
// be zero.  *launched = false if the swarm needs more workgroups than can be
// co-resident (nothing is enqueued then).
hipError_t launch64_gang(int fitness, const Swarm64Args &a, long long T, hipStream_t stream, bool *launched);

// The resident gang (pso_gang64.hip): a whole run by co-resident workgroups
// that hold the swarm in registers; see pso_gang.hpp for the binary32 form.
struct Gang64Args {
    uint32_t T;                // iterations of the launch (at most GANG_MAX_T)
    uint32_t P, L;             // particles per part, lanes per particle
    float block_ratio;         // a meeting's time over an iteration's
    double c1s, c2s;           // c1 2^-24, c2 2^-24 (exact)
    unsigned long long *words; // the parts' meeting words
};
struct Gang64Shape {
    const void *fn;
    int C;
    uint32_t P, L, G, lanes;
    size_t lds;
};
constexpr int GANG64_MAX_D_ALL = 512; // no instantiation holds more dimensions
bool gang64_accepts(int fitness, const Swarm64Args &a);
bool gang64_shape(int fitness, const Swarm64Args &a, int64_t t0, int64_t T, Gang64Shape *out);
size_t gang64_words(uint64_t N, int D); // 64-bit words reserved in the swarm's memory
// What a run returns, as k_fetch64 writes it to pinned host memory; the gbest
// position (D doubles) follows.
struct Fetch64 {
    Ctrl64 ctrl;
    double value;
    double pad[31];
};
hipError_t launch64_fetch(const Swarm64Args &a, Fetch64 *out, hipStream_t stream);
hipError_t launch64_gang_arm(const Swarm64Args &a, hipStream_t stream);
hipError_t launch_gang64(int fitness, const Swarm64Args &a, const Gang64Shape &s, uint32_t T, hipStream_t stream);

} // namespace pso
