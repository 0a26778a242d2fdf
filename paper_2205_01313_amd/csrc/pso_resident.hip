// pso_resident.hip -- the batched kernel whose parts hold their particles in
// vector registers (shape STAGE_REGISTERS).
//
// The LDS-staged batched kernel spends 107 vector instructions per
// particle-dimension update, a third of them on moving the state between LDS
// and registers, item addressing and parameters kept per lane, and one
// 1024-lane workgroup fills a compute unit, which idles whenever that
// workgroup waits: at its barriers, in the fold, for the other parts.  Here a
// workgroup of 256 lanes runs a part: L lanes share a particle, lane k holding
// x, v and p of dimensions [k cs, (k+1) cs), cs <= 16, in registers for the
// whole launch, so an update is 45 to 60 instructions; every parameter of the
// swarm is scalar; and four workgroups share a compute unit, each computing
// while another waits.  What crosses lanes is each particle's fitness: the
// lanes of chunk 0 add their terms in registers, the other chunks stage theirs
// in LDS and the chunk-0 lane adds them in dimension order, the sum of every
// other path.
//
// The parts of a swarm meet once per iteration through tagged words, as in
// the LDS-staged kernel (relaxed device-scope atomics, no fence), each part's
// on a 64-byte line of its own: the step (24 bits) and its best candidate's
// fitness order bits in one word, the candidate's index in a second and its
// position in tagged words read only from the winner.  Parts own ascending
// index ranges, so the lowest part among equal fitness holds the lowest index.
// Deadlock freedom is the work queue's (the grid is co-resident, parts are
// dequeued in order); every wait is bounded.
//
// A part posts its candidate as soon as it has it and computes the own half of
// the next iteration's Eq. 1 (Philox, w v + c1 r1 (p - x)) while the others
// post; the wavefronts in that half yield issue slots to those in the other
// one, on which some swarm's parts wait (s_setprio).
//
// Bound by vector instruction issue (62 instructions per update, 65 % of the
// issue slots on the batch below) and by the slowest of a swarm's parts.  256
// swarms of 32 to 8192 particles, D = 2 to 64, 500 iterations: 30.4 ms
// LDS-staged; here 19.7 with the whole update between the meetings, 18.6 with
// the own half ahead, 17.9 with its priority lowered.  Four workgroups of 256
// lanes rather than one of 1024: the other three compute through one's
// meeting.  16 dimensions per lane: 48 state registers of 128 (c2 r2 of the
// own half waits in the lane's LDS terms), and no shape of the range needs more
// than four lanes per particle.  With the five functions in one kernel 27 vector
// and 482 scalar registers spill.
#include <algorithm>

#include "pso_block.hpp"
#include "pso_gang_device.hpp"
#include "pso_quad.hpp"

namespace pso {

namespace {

constexpr int C = RESIDENT_C, LANES = RESIDENT_LANES;
constexpr int CP = C + 1; // odd stride of a lane's staged terms
constexpr unsigned long long WAIT_TICKS = 2000000000ull; // 20 s of the 100 MHz wall clock
constexpr unsigned long long NONE40 = 0xFFFFFFFFFFull;

struct Shared {
    unsigned long long comb[3]; // a step's best candidate: order bits << 16 | particle of the part; slots in turn
    unsigned long long win;     // the meeting's result: order bits << 12 | part, ~0 if none
    uint32_t win_idx, err, idx;
};

// What a wavefront loads from memory at an address that is the same in every
// lane, in a scalar register.
template <class T>
__device__ __forceinline__ T uniform(T v)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "whole registers");
    uint32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (unsigned q = 0; q < sizeof(T) / 4; ++q) w[q] = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[q]);
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

// Waits until *w carries tag in the bits above `shift`.
__device__ __forceinline__ unsigned long long tagged(const unsigned long long *w, unsigned long long tag, int shift,
                                                     unsigned long long t0, Shared &sh)
{
    unsigned long long v;
    for (uint32_t spins = 0;
         ((v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> shift) != tag;) {
        __builtin_amdgcn_s_sleep(1); // other workgroups of the compute unit have work
        if ((++spins & 63u) == 0u && wall_clock64() - t0 > WAIT_TICKS) {
            sh.err = 1u;
            break;
        }
    }
    return v;
}

template <int FIT>
__device__ __forceinline__ void resident_part(const BatchItem &item, const BatchEntry e, BatchResult *res,
                                              long long chunk, long long iter_cap, float *lds, Shared &sh,
                                              BatchResult *out_state, float *out_pos, int pos_stride)
{
    constexpr int W = Fitness<FIT>::STAGE_WORDS, CW = W * CP;
    // the swarm's fields, scalar
    float *const gx = uniform(item.a.x), *const gv = uniform(item.a.v), *const gp = uniform(item.a.p);
    float *const gpf = uniform(item.a.pf), *const ggpos = uniform(item.a.gpos);
    uint8_t *const gpend = uniform(item.a.pend);
    const float *const gshift = uniform(item.a.shift);
    const uint32_t N = uniform(item.a.N), Np = uniform(item.a.Np), k0 = uniform(item.a.k0), k1 = uniform(item.a.k1);
    const int D = uniform(item.a.D);
    const float lo = uniform(item.a.lo), hi = uniform(item.a.hi), w = uniform(item.a.w), vmax = uniform(item.a.vmax);
    const float c1s = uniform(item.a.c1) * 0x1p-24f, c2s = uniform(item.a.c2) * 0x1p-24f; // exact (short_forms_exact)
    const uint32_t parts = uniform(item.parts), part = e.part;
    const float tol = uniform(item.tol), fstar = uniform(item.fstar);
    unsigned long long *const kw = uniform(item.cand_key);
    unsigned long long *const pw = reinterpret_cast<unsigned long long *>(uniform(item.cand_pos));
    const ResidentSplit R = resident_split(N, D);
    const uint32_t P = R.P, tid = threadIdx.x;
    const int L = (int)R.L, cs = (int)R.cs;
    const int k = __builtin_amdgcn_readfirstlane((int)(tid / P)); // P is a multiple of 64
    const uint32_t j = tid - (uint32_t)k * P, base = part * P, i = base + j;
    const int d0 = k * cs, nd = k < L ? min(cs, D - d0) : 0;
    const bool valid = k < L && i < N, folder = valid && k == 0;
    float *s_g = lds, *s_shift = lds + RESIDENT_MAX_D;
    float *s_t = s_shift + RESIDENT_MAX_D, *s_last = s_t + CW * LANES;
    uint32_t *s_imp = reinterpret_cast<uint32_t *>(s_last + (LANES - P));
    float *my_t = s_t + tid * CW;

    const bool started = uniform(res->started) != 0u;
    unsigned long long gkey = started ? uniform(res->gkey) : NO_KEY;
    long long giter = started ? uniform(res->giter) : 0, t = started ? uniform(res->iters) : -1;
    bool stop = started && uniform(res->stop) != 0u;
    for (int d = (int)tid; d < L * cs; d += LANES) {
        s_g[d] = started && d < D ? ggpos[d] : 0.0f;
        s_shift[d] = d < D ? gshift[d] : 0.0f;
    }
    if (tid < 3) sh.comb[tid] = ~0ull;
    float x[C], v[C], p[C], pf = -__builtin_inff();
#pragma unroll
    for (int q = 0; q < C; ++q) x[q] = v[q] = p[q] = 0.0f;
    if (started && valid) {
        const bool pend = gpend[i] != 0;
#pragma unroll
        for (int q = 0; q < C; ++q) {
            if (q < nd) {
                const size_t at = (size_t)(d0 + q) * Np + i;
                x[q] = gx[at];
                v[q] = gv[at];
                p[q] = pend ? x[q] : gp[at];
            }
        }
        if (folder) pf = gpf[i];
    }
    __syncthreads();

    // iterations this launch: about `chunk` particle-dimension updates' worth
    // (at least one); the same number for every part of the swarm
    const long long done0 = started ? t : 0, left = uniform(item.max_iter) - done0;
    long long iters = chunk / ((long long)N * D);
    iters = iters < 1 ? 1 : (iters > iter_cap ? iter_cap : iters);
    if (e.iters > 0) iters = e.iters;
    iters = left < iters ? left : iters;
    const long long t_end = done0 + iters;
    auto meets = [&]() { return tol > 0.0f && __builtin_fabsf(key_fitness(gkey) - fstar) < tol; };
    stop = stop || (started && meets());
    const unsigned long long c0 = wall_clock64();
    // Step 0 is Step 1 (Alg. 1), step t > 0 iteration t.  A pass of the loop:
    // the social half of Eq. 1, Eq. 2, the fitness, Steps 4 and 5's candidate
    // and its posting (not on a resumed launch's first pass); the own half of
    // the next step's Eq. 1, while the other parts post; the meeting.
    // v holds its own half meanwhile, the first words of the lane's terms c2 r2
    bool skip = started;
    while (!stop) {
        const uint32_t step = (uint32_t)(t + 1);
        unsigned long long comb = ~0ull;
        bool mine = false, imp = false;
        int ndo = nd, ko = k;
        asm volatile("" : "+s"(ndo), "+s"(ko)); // scalar compares in the loop, not masks kept across it
        if (!skip) {
            const bool init = step == 0u;
            Fitness<FIT> fit;
            float zp = 0.0f;
#pragma unroll
            for (int q = 0; q < C; q += 2) {
                if (q >= ndo) continue;
                float w0[2], w1[2] = {0.0f, 0.0f};
                if (init) {
                    const U4 u = philox4x32_10(k0, k1, (uint32_t)(d0 + q) >> 1, i, 0u, TAG_INIT);
                    const float span = hi - lo, vspan = vmax + vmax;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        x[q + h] = clampf(lo + span * unit_float(word_r1(u, h)), lo, hi);
                        v[q + h] = clampf(-vmax + vspan * unit_float(word_r2(u, h)), -vmax, vmax);
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const float nv = clamp_sym(v[q + h] + (my_t[q + h] * (s_g[d0 + q + h] - x[q + h])), vmax);
                        v[q + h] = nv;
                        x[q + h] = clamp_pos(x[q + h] + nv, lo, hi);
                    }
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float z = x[q + h] - s_shift[d0 + q + h];
                    if constexpr (FIT == F_ROSENBROCK) {
                        // a chunk's first term needs the previous chunk's z
                        w0[h] = q + h == 0 ? z : rosen_term(z, zp);
                    } else {
                        w0[h] = gang_term<FIT>(z);
                        if constexpr (W == 2) w1[h] = cos2pi_small(z);
                    }
                    zp = z;
                }
                if (ko > 0) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        my_t[q + h] = w0[h];
                        if constexpr (W == 2) my_t[CP + q + h] = w1[h];
                    }
                } else {
                    if (FIT != F_ROSENBROCK || q > 0) fit.acc = fit.acc + w0[0];
                    if constexpr (W == 2) fit.aux = fit.aux + w1[0];
                    if (q + 1 < ndo) {
                        fit.acc = fit.acc + w0[1];
                        if constexpr (W == 2) fit.aux = fit.aux + w1[1];
                    }
                }
            }
            if (L > 1) { // uniform
                if (FIT == F_ROSENBROCK && k < L - 1) s_last[(uint32_t)k * P + j] = zp;
                __syncthreads();
                if (folder) {
                    for (int kk = 1; kk < L; ++kk) {
                        const float *r = s_t + ((uint32_t)kk * P + j) * CW;
                        const int n = min(cs, D - kk * cs);
#pragma unroll
                        for (int q0 = 0; q0 < C; q0 += 8) {
                            if (q0 >= n) break;
                            float b0[8], b1[8];
#pragma unroll
                            for (int q = 0; q < 8; ++q) {
                                b0[q] = r[q0 + q];
                                b1[q] = W == 2 ? r[CP + q0 + q] : 0.0f;
                            }
                            if (FIT == F_ROSENBROCK && q0 == 0) b0[0] = rosen_term(b0[0], s_last[(uint32_t)(kk - 1) * P + j]);
#pragma unroll
                            for (int q = 0; q < 8; ++q) {
                                if (q0 + q >= n) break;
                                fit.acc = fit.acc + b0[q];
                                if constexpr (W == 2) fit.aux = fit.aux + b1[q];
                            }
                        }
                    }
                }
            }
            // Step 4 (strict; NaN never improves), or every particle at Step 1
            const uint32_t slot = step % 3;
            if (ko == 0) {
                const float f = fit.value(D);
                imp = (init && folder) || f < pf;
                if (imp) {
                    pf = f;
                    const unsigned long long key = make_key(f, i);
                    if (key < gkey) atomicMin(&sh.comb[slot], (key >> 32 << 16) | j);
                }
                if (L > 1 && k == 0) s_imp[j] = imp ? 1u : 0u;
            }
            __syncthreads();
            comb = sh.comb[slot];
            if (tid == 0) sh.comb[(slot + 2) % 3] = ~0ull; // the step after next's; its last readers passed the barrier
            if (L > 1) imp = k < L && s_imp[j] != 0u;
            if (init) imp = valid;
            if (imp) {
#pragma unroll
                for (int q = 0; q < C; ++q) p[q] = x[q];
            }
            // Step 5: the part's candidate
            mine = comb != ~0ull && valid && j == (uint32_t)(comb & 0xFFFFu);
            if (parts > 1) {
                const uint32_t seq = step + 1, par = seq & 1;
                const unsigned long long ptag = (unsigned long long)seq << 32;
                unsigned long long *const line = kw + ((size_t)par * parts + part) * RESIDENT_LINE;
                if (mine) {
                    unsigned long long *dst = pw + ((size_t)par * parts + part) * D + d0;
#pragma unroll
                    for (int q = 0; q < C; ++q)
                        if (q < nd)
                            __hip_atomic_store(&dst[q], ptag | __float_as_uint(x[q]), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                    if (k == 0) __hip_atomic_store(line + 1, ptag | i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (tid == 0)
                    __hip_atomic_store(line, ((unsigned long long)(seq & 0xFFFFFFu) << 40) | (comb == ~0ull ? NONE40 : comb >> 16),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            t = (long long)step;
        }
        if (t < t_end) {
            const uint32_t next = (uint32_t)(t + 1);
            __builtin_amdgcn_s_setprio(0); // after the other workgroups' critical halves
#pragma unroll
            for (int q = 0; q < C; q += 2) {
                if (q >= ndo) continue;
                const U4 u = philox4x32_10(k0, k1, (uint32_t)(d0 + q) >> 1, i, next, TAG_VEL);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float r1 = (float)(word_r1(u, h) >> 8), r2 = (float)(word_r2(u, h) >> 8);
                    v[q + h] = (w * v[q + h]) + ((c1s * r1) * (p[q + h] - x[q + h]));
                    my_t[q + h] = c2s * r2;
                }
            }
        }
        __builtin_amdgcn_s_setprio(3);
        if (skip) {
            skip = false;
            if (t >= t_end) break;
            continue;
        }
        // Step 5: the meeting
        unsigned long long win = comb == ~0ull ? ~0ull : comb >> 16 << 12;
        uint32_t win_idx = base + (uint32_t)(comb & 0xFFFFu);
        if (parts > 1) {
            const uint32_t seq = step + 1, par = seq & 1;
            if (tid < 64) {
                const unsigned long long w0 = wall_clock64();
                unsigned long long best = ~0ull;
                for (uint32_t b = tid; b < parts; b += 64) {
                    const unsigned long long m =
                        tagged(kw + ((size_t)par * parts + b) * RESIDENT_LINE, seq & 0xFFFFFFu, 40, w0, sh) & NONE40;
                    if (m != NONE40) {
                        const unsigned long long c = (m << 12) | b;
                        best = c < best ? c : best;
                    }
                }
                const unsigned long long have = __ballot(best != ~0ull);
                if (have) {
                    if ((have & (have - 1)) == 0) {
                        const int l = __builtin_ctzll(have);
                        best = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(best >> 32), l) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((uint32_t)best, l);
                    } else {
                        best = wave_min_u64(best);
                    }
                    const uint32_t owner = (uint32_t)(best & 0xFFFu);
                    if (tid < (uint32_t)D) // D <= 64
                        s_g[tid] = __uint_as_float(
                            (uint32_t)tagged(pw + ((size_t)par * parts + owner) * D + tid, seq, 32, w0, sh));
                    const uint32_t idx =
                        (uint32_t)tagged(kw + ((size_t)par * parts + owner) * RESIDENT_LINE + 1, seq, 32, w0, sh);
                    if (tid == 0) sh.win_idx = idx;
                }
                if (tid == 0) sh.win = best;
            }
            __syncthreads();
            win = sh.win;
            win_idx = sh.win_idx;
        } else if (comb != ~0ull) { // uniform
            if (mine) {
#pragma unroll
                for (int q = 0; q < C; ++q)
                    if (q < nd) s_g[d0 + q] = x[q];
            }
            __syncthreads();
        }
        if (win != ~0ull) {
            gkey = (win >> 12 << 32) | win_idx;
            giter = t;
        }
        stop = meets();
        if (sh.err || t >= t_end) break; // uniform: err was written before the barrier; the host is told
    }
    const unsigned long long ticks = wall_clock64() - c0;
    if (valid) {
#pragma unroll
        for (int q = 0; q < C; ++q) {
            if (q < nd) {
                const size_t at = (size_t)(d0 + q) * Np + i;
                gx[at] = x[q];
                gv[at] = v[q];
                gp[at] = p[q];
            }
        }
        if (folder) {
            gpf[i] = pf;
            gpend[i] = 0;
        }
    }
    if (part == 0) {
        for (int d = (int)tid; d < D; d += LANES) {
            ggpos[d] = s_g[d];
            if (out_pos) out_pos[(size_t)e.out * pos_stride + d] = s_g[d];
        }
        if (tid == 0) {
            res->gkey = gkey;
            res->giter = giter;
            res->iters = t;
            res->stop = stop ? 1u : 0u;
            res->started = 1u;
            res->ticks = ticks > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)ticks;
            if (out_state) out_state[e.out] = *res;
        }
    }
}

} // namespace

// 128 registers a lane, so four workgroups share a compute unit.
__global__ void __launch_bounds__(LANES) __attribute__((amdgpu_waves_per_eu(4)))
k_batch_resident(const BatchItem *items, const BatchEntry *entries, BatchResult *results, uint32_t count,
                 unsigned int *next, long long chunk, long long iter_cap, BatchResult *out_state, float *out_pos,
                 int pos_stride, unsigned int *err)
{
    __shared__ Shared sh;
    extern __shared__ float s_resident[];
    if (threadIdx.x == 0) sh.err = 0;
    for (;;) {
        if (threadIdx.x == 0) sh.idx = atomicAdd(next, 1u);
        __syncthreads();
        const uint32_t n = uniform(sh.idx);
        __syncthreads();
        if (n >= count) break; // uniform: every workgroup leaves once the list is drained
        BatchEntry e = entries[n];
        e.item = uniform(e.item);
        e.part = uniform(e.part);
        e.out = uniform(e.out);
        e.iters = uniform(e.iters);
        const BatchItem &it = items[e.item];
        BatchResult *res = &results[e.item];
        switch (uniform(it.fitness)) {
        case F_SPHERE: resident_part<F_SPHERE>(it, e, res, chunk, iter_cap, s_resident, sh, out_state, out_pos, pos_stride); break;
        case F_RASTRIGIN: resident_part<F_RASTRIGIN>(it, e, res, chunk, iter_cap, s_resident, sh, out_state, out_pos, pos_stride); break;
        case F_ROSENBROCK: resident_part<F_ROSENBROCK>(it, e, res, chunk, iter_cap, s_resident, sh, out_state, out_pos, pos_stride); break;
        case F_ACKLEY: resident_part<F_ACKLEY>(it, e, res, chunk, iter_cap, s_resident, sh, out_state, out_pos, pos_stride); break;
        default: resident_part<F_CUBIC>(it, e, res, chunk, iter_cap, s_resident, sh, out_state, out_pos, pos_stride); break;
        }
        __syncthreads();
        if (sh.err) break; // uniform
    }
    if (threadIdx.x == 0 && sh.err && err) atomicOr(err, 1u);
}

// Gbest position and shift, the terms of the chunks after the first (two words
// for Ackley), their last z and the improvement flags.
size_t resident_lds() { return sizeof(float) * (2 * RESIDENT_MAX_D + (size_t)LANES * 2 * CP + (LANES - 64) + LANES); }

hipError_t launch_batch_resident(const BatchItem *items, const BatchEntry *entries, BatchResult *results, uint32_t count,
                                 unsigned int *next, int grid, long long chunk, long long iter_cap, hipStream_t stream,
                                 BatchResult *out_state, float *out_pos, int pos_stride, unsigned int *err)
{
    hipLaunchKernelGGL(k_batch_resident, dim3(grid), dim3(LANES), resident_lds(), stream, items, entries, results, count,
                       next, chunk, iter_cap, out_state, out_pos, pos_stride, err);
    return hipGetLastError();
}

hipError_t resident_occupancy(int *per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k_batch_resident, LANES, resident_lds());
}

} // namespace pso
