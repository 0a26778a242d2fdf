// pso_gang.hip -- the resident gang: a whole pso_run of one synchronous swarm
// by co-resident workgroups that keep the swarm in vector registers.
//
// A launch per iteration costs 5 us or more before it does any work, and a
// state of a few megabytes fits the chip's registers (128 MiB), so the
// iteration loop runs inside the workgroups ("parts"): each owns P
// consecutive particles, and L = ceil(D / C) lanes share a particle, lane k
// holding x, v and p of dimensions [k C, (k+1) C) in registers from the first
// iteration to the last.  What a part needs from the others is the gbest
// alone, so all parts meet once per iteration (below).
//
// Lane k * P + j of a part holds chunk k of particle j.  With P a multiple of
// 64 (UNI) a wavefront holds one chunk, so the dimension, its Philox counter
// word and the bounds tests are scalar.  The fitness is a sequential sum over
// the dimensions: the lanes of chunk 0 add their own terms in registers; the
// other chunks stage theirs in LDS and after a barrier the chunk-0 lane adds
// them in dimension order, so the sum is the other paths' bit for bit.  With
// one lane per particle (L = 1) nothing is staged.
//
// Meeting.  Every part posts one 64-bit word per meeting, on a 64-byte line
// of its own: the meeting's number (24 bits), and its best candidate -- a
// particle that beats the gbest -- as (iteration within the meeting's block,
// order bits of the fitness); the candidate's index and position are in tagged
// words beside it that only the winner's readers read.  Parts own ascending
// index ranges, so the lowest part among equal words holds the lowest index.
// Words move by relaxed device-scope atomics, which are coherent per word; no
// fence and no other memory passes between parts.  Measured, all parts of a
// meeting on their own compute unit: 0.87 us (2 parts), 1.1 (64), 1.35 (128),
// 2.2 (248); with the words packed instead of one per line 1.8 at 64 parts.
// While the words travel, the lanes compute the gbest-independent half of the
// next iteration (Philox, inertia and cognitive terms).
//
// Blocks of iterations (SPEC).  Once a swarm of few dimensions has settled
// its gbest changes rarely, and an iteration that changes nothing needs no
// meeting: with the gbest unchanged, particles do not interact.  So a meeting
// covers a block of up to K iterations run ahead with the gbest of the
// block's start.  A wavefront (a part where lanes share particles) stops at
// its first candidate.  The parts agree on the earliest iteration j that has
// one (the least word); whoever ran past j restores the block's start from a
// copy in registers and repeats j iterations.  What is committed is exactly
// the synchronous method's trajectory.  A block costs a meeting M and, when the
// gbest changes in it, about K iterations I run in vain or again; with a
// change every m iterations that is least at K = sqrt(m M / I) (next_block: m
// a running mean, M / I from the shape, block_ratio).  A swarm whose gbest
// changes every iteration meets every iteration (K = 1: no copy, nothing
// repeated).
//
// All parts must be resident together.  They meet once before they touch any
// state; if they are not all there within RENDEZVOUS_TICKS (another kernel
// holds compute units), all leave, the control block says so and the caller
// takes the step launches instead.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "pso_gang.hpp"
#include "pso_gang_device.hpp"
#include "pso_quad.hpp"

namespace pso {

constexpr unsigned long long NO_COMB = ~0ull;

// A lane's chunk; of p, the first C - PL dimensions (the others are in LDS).
template <int C, int PL>
struct LaneState {
    float x[C], v[C], p[C > PL ? C - PL : 1];
    float pf;       // pbest fitness (folding lanes; -inf where there is no particle)
    uint32_t n_imp; // pbest improvements
};

template <int C>
struct OwnHalf { // of the next iteration: (w v) + ((c1 r1)(p - x)) and c2 r2
    float own[C], soc[C];
};

// c1 r1 with r1 = u 2^-24, u an integer below 2^24, is one rounding of the
// product c1 u 2^-24; with c1 2^-24 exact (gang_accepts) so is (c1 2^-24) u.
template <int C>
__device__ __forceinline__ void own_half(const SwarmArgs &a, const GangArgs &ga, int D, int d0, uint32_t i,
                                         uint32_t t, const LaneState<C, 0> &S, OwnHalf<C> &O)
{
    constexpr int Q = group_of(C);
    asm volatile("" : "+s"(D)); // as in the update: no hoisted masks
#pragma unroll
    for (int e = 0; e < C; e += Q) {
        if (d0 + e >= D) continue;
#pragma unroll
        for (int c = e; c < e + Q; c += 2) {
            const U4 u = philox4x32_10(a.k0, a.k1, (uint32_t)(d0 + c) >> 1, i, t, TAG_VEL);
#pragma unroll
            for (int h = 0; h < (C == 1 ? 1 : 2); ++h) {
                const float r1 = (float)(word_r1(u, h) >> 8), r2 = (float)(word_r2(u, h) >> 8);
                O.own[c + h] = (a.w * S.v[c + h]) + ((ga.c1s * r1) * (S.p[c + h] - S.x[c + h]));
                O.soc[c + h] = ga.c2s * r2;
            }
        }
    }
}

// The least of a wavefront's candidates into *least, called by the lanes that
// have one.  A swarm on its way down has many at once, and atomics of one
// address take their turns (Cubic D = 32, N = 64, whose particles improve
// together: 50 iterations 218 us, 155 with one atomic a wavefront).  A candidate
// that beats the one in hand takes its place until none does: fewer rounds than
// a butterfly has for the few there are, and nothing where there is none.
__device__ __forceinline__ void post_least(unsigned long long *least, unsigned long long comb)
{
    const uint32_t lo = (uint32_t)comb, hi = (uint32_t)(comb >> 32);
    unsigned long long best = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)hi) << 32) |
                              (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
    while (const unsigned long long m = __ballot(comb < best)) {
        const int l = __builtin_ctzll(m);
        best = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)hi, l) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)lo, l);
    }
    if (comb == best) atomicMin(least, best); // one lane: particles differ
}

struct GangShared {
    unsigned long long comb[3]; // a block's best candidate: j << 48 | order bits << 16 | particle of the part
    unsigned long long win;     // the meeting's result: low 40 bits of the winner's word << 8 | part, NO_COMB if none
    uint32_t win_idx;
    uint32_t err, go;
};

// PL: dimensions of p kept in LDS, the last of the chunk (large chunks: x, v
// and p of 64 dimensions are 192 registers of the 256 a lane has at 512 lanes).
// Several forms spill all the same: at 1024 lanes (128 registers) C = 16 23 to 63
// registers and C = 8 without whole wavefronts 12 to 20, C = 32 and 64 10 to 22; the
// shapes below were measured with that.  TAIL (Ackley in two chunks of 64: its two words of terms and
// p do not both fit LDS): chunk 1's lanes keep their cosines in LDS, and after
// the barrier continue chunk 0's two sums themselves, their z^2 from x.
template <int FIT, int C, bool MULTI, bool UNI, bool SPEC, int MAXT, int PL = 0, bool TAIL = false>
__global__ void __launch_bounds__(MAXT) k_gang_resident(SwarmArgs a, GangArgs ga)
{
    constexpr int W = Fitness<FIT>::STAGE_WORDS;
    constexpr int Q = group_of(C), PR = C - PL, FK = TAIL ? 1 : 0; // FK: the chunk whose lanes fold
    constexpr bool STAGE = MULTI && !TAIL;
    static_assert((C == 1 && !MULTI) || C % 2 == 0, "chunks hold whole Philox pairs");
    static_assert(!TAIL || (MULTI && FIT == F_ACKLEY), "one word of two recomputed");
    __shared__ GangShared sh;
    // gbest position (two of them: a repeated block still reads the old one)
    // and shift (L * C floats each), then with MULTI the staged terms of the
    // chunks after the first -- a lane's are CP floats apart, word after word,
    // C + 1 of them so that consecutive lanes start on different banks and
    // every address is one register plus a constant --, each chunk's last z
    // (Rosenbrock), the improvement flags, and p's PL dimensions of each lane
    extern __shared__ float s_gang[];
    Ctrl *c = a.ctrl;
    const int D = a.D;
    const uint32_t P = ga.P, G = gridDim.x, part = blockIdx.x, tid = threadIdx.x, T = blockDim.x;
    const int L = (int)ga.L, DL = L * C;
    float *s_gpos = s_gang, *s_shift = s_gang + 2 * DL;
    constexpr int CP = C + 1, CW = W * CP;
    float *s_t = s_shift + DL, *s_last = s_t + (STAGE ? (size_t)CW * (L - 1) * P : TAIL ? (size_t)(CP + 2) * P : 0);
    uint32_t *s_imp = reinterpret_cast<uint32_t *>(s_last + (FIT == F_ROSENBROCK ? (size_t)(L - 1) * P : 0));
    float *my_p = reinterpret_cast<float *>(s_imp + (MULTI ? P : 0)) + tid * (PL + 1); // odd stride: no bank conflicts
    int k_lane = MULTI ? (int)(tid / P) : 0;
    if (UNI) k_lane = __builtin_amdgcn_readfirstlane(k_lane);
    const int k = k_lane;
    const uint32_t j = MULTI ? tid - (uint32_t)k * P : tid;
    const int d0 = k * C;
    const uint32_t base = part * P, i = base + j;
    const bool valid = j < P && k < L && i < a.N;
    const bool folder = valid && k == FK;

    // control block, before any part can write it back
    unsigned long long gkey = c->gkey_prev;
    long long giter = c->giter;
    const long long t0 = c->t;
    bool stop = c->stop != 0u;
    const float tol = c->tol, fstar = c->fstar;

    // this part's meeting words (both parities) to zero, then the rendezvous
    unsigned long long *const kw = ga.words, *const pw = ga.words + (size_t)2 * KEY_STRIDE * G;
    const uint32_t pstride = (uint32_t)D;
    if (G > 1) {
        for (uint32_t q = tid; q < 2 * (2 + pstride); q += T) {
            const uint32_t par = q & 1, w = q >> 1;
            unsigned long long *dst = w < 2 ? kw + ((size_t)par * G + part) * KEY_STRIDE + w
                                            : pw + ((size_t)par * G + part) * pstride + (w - 2);
            __hip_atomic_store(dst, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    for (int d = (int)tid; d < DL; d += (int)T) {
        s_gpos[d] = d < D ? a.gpos[d] : 0.0f;
        s_shift[d] = d < D ? a.shift[d] : 0.0f;
    }
    if (tid < 3) sh.comb[tid] = NO_COMB;
    if (tid == 0) sh.err = 0;
    __syncthreads();
    if (G > 1) {
        if (tid == 0) {
            __threadfence(); // the zeroed words precede the arrival
            if (atomicAdd(&c->gang_arrive, 1u) == G - 1) atomicCAS(&c->gang_state, 0u, GANG_GO);
            const unsigned long long w0 = wall_clock64();
            uint32_t st;
            while ((st = __hip_atomic_load(&c->gang_state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0u) {
                __builtin_amdgcn_s_sleep(1);
                // whichever of GO and ABSENT is set first holds for every part
                if (wall_clock64() - w0 > RENDEZVOUS_TICKS) atomicCAS(&c->gang_state, 0u, GANG_ABSENT);
            }
            sh.go = st == GANG_GO;
        }
        __syncthreads();
        if (!sh.go) return; // uniform; no state was touched
    }

    LaneState<C, PL> S;
    S.pf = -__builtin_inff();
    S.n_imp = 0;
    {
        const bool pend = valid && a.pend[i] != 0;
#pragma unroll
        for (int e = 0; e < C; ++e) {
            float pe = 0.0f;
            S.x[e] = S.v[e] = 0.0f;
            if (valid && d0 + e < D) {
                const size_t at = (size_t)(d0 + e) * a.Np + i;
                S.x[e] = a.x[at];
                S.v[e] = a.v[at];
                pe = pend ? S.x[e] : a.p[at];
            }
            if (e < PR) S.p[e < PR ? e : 0] = pe;
            else my_p[e - PR] = pe;
        }
        if (folder) S.pf = a.pf[i];
    }
    // every lane of a particle has read its mark before the folding lane clears
    // it: a launch whose stop rule already holds meets no other barrier
    if constexpr (MULTI) __syncthreads();

    float *s_g = s_gpos, *s_gn = s_gpos + DL; // in use, and the next one
    constexpr bool AHEAD = C <= 16 && PL == 0; // room for the next iteration's own half in registers
    OwnHalf<AHEAD ? C : 1> O;
    bool have_own = false;

    // Steps 2-4 of iteration t; cand: this lane's particle improved and beats
    // the gbest, with fitness order bits ord
    auto iterate = [&](uint32_t t, int slot, bool collect, bool &cand, uint32_t &ord) {
        // opaque copies: the tests on them are scalar compares here, instead of
        // masks computed once before the loop and spilled
        int D = a.D, k = k_lane;
        asm volatile("" : "+s"(D));
        if constexpr (UNI) asm volatile("" : "+s"(k));
        const int d0 = k * C;
        Fitness<FIT> fit;
        float zp = 0.0f; // previous dimension's z (Rosenbrock)
        float *my_t = s_t + (STAGE && k > 0 ? (tid - P) * CW : TAIL ? 2 * P + j * CP : 0u);
        if constexpr (AHEAD) {
            if (!have_own) own_half<C>(a, ga, D, d0, i, t, S, O);
            have_own = false;
        }
#pragma unroll
        for (int e = 0; e < C; e += Q) {
            // large chunks: no scheduling across groups (their loads and draws
            // in flight together would not fit the registers)
            if constexpr (!AHEAD) __builtin_amdgcn_sched_barrier(0);
            if (d0 + e >= D) continue;
            float w0[Q], w1[W == 2 ? Q : 1];
#pragma unroll
            for (int q = e; q < e + Q; q += 2) {
                U4 u{};
                if constexpr (!AHEAD) u = philox4x32_10(a.k0, a.k1, (uint32_t)(d0 + q) >> 1, i, t, TAG_VEL);
#pragma unroll
                for (int h = 0; h < (C == 1 ? 1 : 2); ++h) {
                    const int c = q + h, d = d0 + c;
                    float own, soc;
                    if constexpr (AHEAD) {
                        own = O.own[c];
                        soc = O.soc[c];
                    } else {
                        const float r1 = (float)(word_r1(u, h) >> 8), r2 = (float)(word_r2(u, h) >> 8);
                        const float pc = c < PR ? S.p[c < PR ? c : 0] : my_p[c - PR];
                        own = (a.w * S.v[c]) + ((ga.c1s * r1) * (pc - S.x[c]));
                        soc = ga.c2s * r2;
                    }
                    const float nv = clamp_sym(own + (soc * (s_g[d] - S.x[c])), a.vmax);
                    const float xn = clamp_pos(S.x[c] + nv, a.lo, a.hi);
                    S.v[c] = nv;
                    S.x[c] = xn;
                    const float z = xn - s_shift[d];
                    if constexpr (FIT == F_ROSENBROCK) {
                        // a chunk's first term needs the previous chunk's z
                        w0[c - e] = c == 0 ? z : rosen_term(z, zp);
                    } else {
                        w0[c - e] = gang_term<FIT>(z);
                        if constexpr (W == 2) w1[c - e] = cos2pi_small(z);
                    }
                    zp = z;
                }
            }
            if constexpr (TAIL) {
                if (k == 1) {
#pragma unroll
                    for (int c = 0; c < Q; ++c) my_t[e + c] = w1[c];
                    continue;
                }
            }
            if (STAGE && k > 0) {
#pragma unroll
                for (int c = 0; c < Q; ++c) {
                    my_t[e + c] = w0[c];
                    if constexpr (W == 2) my_t[CP + e + c] = w1[c];
                }
            } else {
                // summed in registers (Rosenbrock has no term for d = 0)
#pragma unroll
                for (int c = 0; c < Q; ++c) {
                    if (c > 0 && d0 + e + c >= D) break;
                    if (FIT != F_ROSENBROCK || e + c > 0) fit.acc = fit.acc + w0[c];
                    if constexpr (W == 2) fit.aux = fit.aux + w1[c];
                }
            }
            if (MULTI && FIT == F_ROSENBROCK && e == C - Q && k < L - 1) s_last[(uint32_t)k * P + j] = zp;
        }
        if constexpr (TAIL) {
            if (k == 0 && j < P) {
                s_t[j] = fit.acc;
                s_t[P + j] = fit.aux;
            }
            __syncthreads();
            if (k == 1) {
                fit.acc = s_t[j];
                fit.aux = s_t[P + j];
#pragma unroll
                for (int e = 0; e < C; e += Q) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (d0 + e >= D) continue;
#pragma unroll
                    for (int c = e; c < e + Q; ++c) {
                        if (c > e && d0 + c >= D) break;
                        const float z = S.x[c] - s_shift[d0 + c];
                        fit.acc = fit.acc + z * z;
                        fit.aux = fit.aux + my_t[c];
                    }
                }
            }
        }
        if constexpr (STAGE) {
            __syncthreads();
            if (folder) {
                // a batch of terms is loaded before they are added, so the sum
                // waits on LDS once a batch; terms past D are loaded (their
                // place exists) but not added
                constexpr int MOST = (MAXT <= 512 ? 32 : 16) / W; // terms of a batch
                constexpr int BS = C < MOST ? C : MOST, NB = MOST / BS; // of a chunk, chunks
                for (int kk = 1; kk < L; kk += NB) {
                    const float *r = s_t + ((uint32_t)(kk - 1) * P + j) * CW;
#pragma unroll
                    for (int q0 = 0; q0 < C; q0 += BS) {
                        float b0[NB][BS], b1[NB][W == 2 ? BS : 1], last[NB];
#pragma unroll
                        for (int n = 0; n < NB; ++n) {
                            if (kk + n >= L) break;
#pragma unroll
                            for (int q = 0; q < BS; ++q) {
                                b0[n][q] = r[(uint32_t)n * P * CW + q0 + q];
                                if constexpr (W == 2) b1[n][q] = r[(uint32_t)n * P * CW + CP + q0 + q];
                            }
                            // the chunk's first row holds its z; the term needs
                            // the previous chunk's last
                            if (FIT == F_ROSENBROCK && q0 == 0) last[n] = s_last[(uint32_t)(kk + n - 1) * P + j];
                        }
#pragma unroll
                        for (int n = 0; n < NB; ++n) {
                            if (kk + n >= L) break;
                            if (FIT == F_ROSENBROCK && q0 == 0) b0[n][0] = rosen_term(b0[n][0], last[n]);
#pragma unroll
                            for (int q = 0; q < BS; ++q) {
                                if ((kk + n) * C + q0 + q >= D) break;
                                fit.acc = fit.acc + b0[n][q];
                                if constexpr (W == 2) fit.aux = fit.aux + b1[n][q];
                            }
                        }
                    }
                }
            }
        }
        // Step 4: strict improvement; NaN never improves
        bool imp = false;
        cand = false;
        ord = 0xFFFFFFFFu;
        if (!MULTI || k == FK) {
            const float f = fit.value(D);
            imp = f < S.pf;
            if (imp) {
                S.pf = f;
                ++S.n_imp;
                const unsigned long long key = make_key(f, i);
                cand = key < gkey;
                ord = (uint32_t)(key >> 32);
            }
        }
        if constexpr (MULTI) {
            if (k == FK && j < P) s_imp[j] = imp ? 1u : 0u;
            if (collect && cand) post_least(&sh.comb[slot], (1ull << 48) | ((unsigned long long)ord << 16) | j);
            __syncthreads();
            imp = j < P && s_imp[j] != 0u;
        }
        if (imp) {
#pragma unroll
            for (int q = 0; q < C; ++q) {
                if (q < PR) S.p[q < PR ? q : 0] = S.x[q];
                else my_p[q - PR] = S.x[q];
            }
        }
    };

    long long done = 0;
    int K = 1;
    float mean = 1.0f, since = 0.0f; // iterations between gbest changes, and since the last
    uint32_t seq = 0;
    stop = stop || (tol > 0.0f && __builtin_fabsf(key_fitness(gkey) - fstar) < tol);
    while (done < (long long)ga.T && !stop) {
        ++seq;
        const uint32_t tb = (uint32_t)(t0 + done);
        const int n = SPEC ? (int)min((long long)K, (long long)ga.T - done) : 1;
        int slot = (int)(seq % 3);
        LaneState<SPEC ? C : 1, PL> B;
        if constexpr (SPEC) {
            if (n > 1) B = S;
        }
        // the block: up to n iterations, as far as this wavefront's (part's)
        // first candidate
        int ran = 0;
        bool cand = false;
        uint32_t ord = 0;
        unsigned long long comb;
        if constexpr (MULTI) {
            do {
                ++ran;
                iterate(tb + (uint32_t)ran, slot, true, cand, ord); // ends with a barrier
                comb = sh.comb[slot];
            } while (ran < n && comb == NO_COMB);
            if (comb != NO_COMB) comb += (unsigned long long)(ran - 1) << 48;
        } else {
            bool any;
            do {
                ++ran;
                iterate(tb + (uint32_t)ran, slot, false, cand, ord);
                any = __any(cand);
            } while (ran < n && !any);
            if (cand) post_least(&sh.comb[slot], ((unsigned long long)ran << 48) | ((unsigned long long)ord << 16) | j);
            __syncthreads();
            comb = sh.comb[slot];
        }
        // the slot of the block after the next; its last readers (the block
        // before) passed the barrier above
        if (tid == 0) sh.comb[(slot + 2) % 3] = NO_COMB;
        unsigned long long win;
        uint32_t win_idx;
        if (G > 1) {
            const uint32_t par = seq & 1;
            const unsigned long long ptag = (unsigned long long)seq << 32;
            if (comb != NO_COMB && valid && j == (uint32_t)(comb & 0xFFFFu)) {
                unsigned long long *dst = pw + ((size_t)par * G + part) * pstride;
#pragma unroll
                for (int q = 0; q < C; ++q)
                    if (d0 + q < D)
                        __hip_atomic_store(&dst[d0 + q], ptag | __float_as_uint(S.x[q]), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                if (k == 0)
                    __hip_atomic_store(kw + ((size_t)par * G + part) * KEY_STRIDE + 1, ptag | i, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
            if (tid == 0)
                __hip_atomic_store(kw + ((size_t)par * G + part) * KEY_STRIDE,
                                   ((unsigned long long)(seq & 0xFFFFFFu) << 40) | ((comb >> 16) & 0xFFFFFFFFFFull),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if constexpr (AHEAD) {
                // meanwhile the next iteration's own half (of a block that
                // cannot be rolled back)
                if (n == 1 && done + 1 < (long long)ga.T) {
                    own_half<C>(a, ga, D, d0, i, tb + 2, S, O);
                    have_own = true;
                }
            }
            if (tid < 64) {
                const unsigned long long w0 = wall_clock64();
                unsigned long long best = NO_COMB;
                const uint32_t want = seq & 0xFFFFFFu;
                unsigned long long v[GANG_PARTS_MAX / 64];
                for (uint32_t spins = 0;;) {
                    bool all = true;
#pragma unroll
                    for (int q = 0; q < (int)GANG_PARTS_MAX / 64; ++q) {
                        const uint32_t b = tid + 64 * q;
                        if (64u * q < G)
                            v[q] = b < G ? __hip_atomic_load(kw + ((size_t)par * G + b) * KEY_STRIDE, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT)
                                         : (unsigned long long)want << 40 | 0xFFFFFFFFFFull;
                    }
#pragma unroll
                    for (int q = 0; q < (int)GANG_PARTS_MAX / 64; ++q)
                        if (64u * q < G) all = all && (v[q] >> 40) == want;
                    if (__all(all)) break;
                    if ((++spins & 63u) == 0u && wall_clock64() - w0 > GANG_TICKS) {
                        sh.err = 1u;
                        break;
                    }
                }
#pragma unroll
                for (int q = 0; q < (int)GANG_PARTS_MAX / 64; ++q) {
                    if (64u * q >= G) continue;
                    const unsigned long long w = v[q] & 0xFFFFFFFFFFull;
                    const unsigned long long m = w == 0xFFFFFFFFFFull ? NO_COMB : (w << 8) | (tid + 64 * q);
                    best = m < best ? m : best;
                }
                const unsigned long long have = __ballot(best != NO_COMB);
                if (have) {
                    if ((have & (have - 1)) == 0) {
                        const int l = __builtin_ctzll(have);
                        best = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(best >> 32), l) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((uint32_t)best, l);
                    } else {
                        best = wave_min_u64(best);
                    }
                    const unsigned long long *src = pw + ((size_t)par * G + (uint32_t)(best & 0xFF)) * pstride;
                    const unsigned long long *srci = kw + ((size_t)par * G + (uint32_t)(best & 0xFF)) * KEY_STRIDE + 1;
                    for (uint32_t q0 = 0; q0 < (uint32_t)D; q0 += 128) {
                        unsigned long long pv[2], pi;
                        for (uint32_t spins = 0;;) {
                            pi = __hip_atomic_load(srci, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                            for (int e = 0; e < 2; ++e) {
                                const uint32_t q = q0 + 64 * e + tid;
                                pv[e] = q < (uint32_t)D
                                            ? __hip_atomic_load(&src[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                            : ptag;
                            }
                            const bool all = (pi >> 32) == seq && (pv[0] >> 32) == seq && (pv[1] >> 32) == seq;
                            if (__all(all)) break;
                            if ((++spins & 63u) == 0u && wall_clock64() - w0 > GANG_TICKS) {
                                sh.err = 1u;
                                break;
                            }
                        }
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const uint32_t q = q0 + 64 * e + tid;
                            if (q < (uint32_t)D) s_gn[q] = __uint_as_float((uint32_t)pv[e]);
                        }
                        if (tid == 0) sh.win_idx = (uint32_t)pi;
                    }
                }
                if (tid == 0) sh.win = best;
            }
            __syncthreads();
            win = sh.win;
            win_idx = sh.win_idx;
            if (sh.err) break; // uniform; the state is lost and the caller told
        } else {
            win = comb == NO_COMB ? NO_COMB : (comb >> 16) << 8;
            win_idx = base + (uint32_t)(comb & 0xFFFFu);
            if (comb != NO_COMB) { // uniform
                if (valid && j == (uint32_t)(comb & 0xFFFFu)) {
#pragma unroll
                    for (int q = 0; q < C; ++q)
                        if (d0 + q < D) s_gn[d0 + q] = S.x[q];
                }
                __syncthreads();
            }
        }
        const bool changed = win != NO_COMB;
        const int nc = changed ? (int)(win >> 40) : n; // iterations committed
        if constexpr (SPEC) {
            // ran past the change: repeat its nc iterations from the block's
            // start, with the gbest of then
            if (changed && ran != nc) {
                S = B;
                for (int s = 1; s <= nc; ++s) iterate(tb + (uint32_t)s, slot, false, cand, ord);
            }
        }
        if (part == 0 && a.hist) {
            for (int s = 1 + (int)tid; s <= nc; s += (int)T)
                a.hist[(tb + (uint32_t)s) & (HIST_CAP - 1)] =
                    changed && s == nc ? (((win >> 8) & 0xFFFFFFFFull) << 32) | win_idx : gkey;
        }
        if (changed) {
            gkey = (((win >> 8) & 0xFFFFFFFFull) << 32) | win_idx;
            giter = t0 + done + nc;
            float *s_old = s_g;
            s_g = s_gn;
            s_gn = s_old;
        }
        done += nc;
        K = SPEC ? next_block(changed, nc, ga.block_ratio, mean, since) : 1;
        stop = tol > 0.0f && __builtin_fabsf(key_fitness(gkey) - fstar) < tol;
    }

#pragma unroll
    for (int e = 0; e < C; ++e) {
        if (valid && d0 + e < D) {
            const size_t at = (size_t)(d0 + e) * a.Np + i;
            a.x[at] = S.x[e];
            a.v[at] = S.v[e];
            a.p[at] = e < PR ? S.p[e < PR ? e : 0] : my_p[e - PR];
        }
    }
    if (folder) {
        a.pf[i] = S.pf;
        a.pend[i] = 0;
    }
    uint32_t n_imp = folder ? S.n_imp : 0u;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) n_imp += __shfl_xor(n_imp, off, 64);
    if ((tid & 63) == 0 && n_imp) atomicAdd(&c->improved, (unsigned long long)n_imp);
    if (tid == 0 && sh.err) atomicOr(&c->err, ERR_GANG_WAIT);
    if (part != 0) return;
    for (int d = (int)tid; d < D; d += (int)T) a.gpos[d] = s_g[d];
    if (tid == 0) {
        c->gkey = gkey;
        c->gkey_prev = gkey;
        c->pubkey = gkey;
        c->giter = giter;
        c->t = t0 + done;
        c->stop = stop ? 1u : 0u;
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
bool gang_accepts(int fitness, const SwarmArgs &a, float shift_max, bool state_set)
{
    const char *env = getenv("PSO_GANG");
    if (env && !strcmp(env, "0")) return false;
    return short_forms_exact(fitness, a.lo, a.hi, a.c1, a.c2, shift_max, state_set);
}

size_t gang_words(uint32_t parts, int D)
{
    return (size_t)2 * parts * KEY_STRIDE + (size_t)2 * parts * (size_t)D;
}

// One instantiation: its kernel, chunk and lane limit.
struct GangKernel {
    const void *fn;
    int C, max_lanes, pl;
    bool multi, uni, tail;
};

template <int FIT, int C, bool MULTI, bool UNI, bool SPEC, int MAXT, int PL = 0, bool TAIL = false>
static GangKernel gang_entry()
{
    return GangKernel{reinterpret_cast<const void *>(k_gang_resident<FIT, C, MULTI, UNI, SPEC, MAXT, PL, TAIL>),
                      C, MAXT, PL, MULTI, UNI, TAIL};
}

template <int FIT>
static const GangKernel *gang_table(int *n)
{
    constexpr bool two = Fitness<FIT>::STAGE_WORDS == 2;
    static const GangKernel t[] = {
        gang_entry<FIT, 1, false, true, true, 1024>(),
        gang_entry<FIT, 2, false, true, true, 1024>(),
        gang_entry<FIT, 4, false, true, true, 1024>(),
        gang_entry<FIT, 8, false, true, true, 512>(),
        gang_entry<FIT, 8, false, true, false, 1024>(),
        gang_entry<FIT, 16, false, true, true, 512>(),
        gang_entry<FIT, 16, false, true, false, 1024>(),
        gang_entry<FIT, 32, false, true, false, 1024, 32>(),
        gang_entry<FIT, 64, false, true, false, 512, 64>(),
        gang_entry<FIT, 2, true, true, true, 1024>(),
        gang_entry<FIT, 4, true, true, true, 1024>(),
        gang_entry<FIT, 8, true, true, false, 1024>(),
        gang_entry<FIT, 16, true, true, false, 1024>(),
        gang_entry<FIT, 2, true, false, true, 1024>(),
        gang_entry<FIT, 4, true, false, true, 1024>(),
        gang_entry<FIT, 8, true, false, false, 1024>(),
        gang_entry<FIT, 64, true, true, false, 512, 32, two>(),
    };
    *n = (int)(sizeof t / sizeof t[0]);
    return t;
}

static const GangKernel *gang_kernels(int fitness, int *n)
{
    switch (fitness) {
    case F_SPHERE: return gang_table<F_SPHERE>(n);
    case F_RASTRIGIN: return gang_table<F_RASTRIGIN>(n);
    case F_ROSENBROCK: return gang_table<F_ROSENBROCK>(n);
    case F_ACKLEY: return gang_table<F_ACKLEY>(n);
    default: return gang_table<F_CUBIC>(n);
    }
}

// Chosen by measurement (us per iteration of the first 200 and of 1000 at
// ratios 0.2 / 1 / 4 / 16): Sphere D = 2, N = 1024 1.86 / 1.64 / 1.48 / 1.65
// and 0.83 / 0.69 / 0.62 / 0.64; Sphere D = 10, N = 5000 (lanes share
// particles) 2.89 / 2.92 / 3.36 / 4.67 and 1.58 / 1.43 / 1.47 / 1.74; Cubic D =
// 1, N = 16384 1.10 / 0.77 / 0.65 / 0.59.  One part whose lanes share
// particles stops as a whole at its first candidate, so nothing is repeated
// and blocks are as long as they may be.
float block_ratio(int C, uint32_t L, uint32_t lanes, uint32_t G, float weight)
{
    if (G == 1 && L > 1) return 1e6f;
    const float meeting = G > 1 ? 1.5f + (float)G / 256.0f : 0.7f;
    const float iteration = 0.15f + 0.1f * weight * (float)C * std::max(1.0f, (float)lanes / 512.0f) + (L > 1 ? 1.2f : 0.0f);
    return meeting / iteration;
}

bool gang_device(int *cus, int *lds)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return false;
    return true;
}

static size_t gang_lds(int fitness, int D, const GangKernel &kn, uint32_t P, uint32_t L)
{
    const size_t lanes = ((size_t)P * L + 63) / 64 * 64;
    size_t f = 3 * (size_t)L * kn.C;
    if (kn.tail) f += (size_t)(kn.C + 3) * P;
    else if (kn.multi) f += (size_t)(fitness == F_ACKLEY ? 2 : 1) * (kn.C + 1) * (L - 1) * P;
    if (kn.multi && fitness == F_ROSENBROCK) f += (size_t)(L - 1) * P;
    if (kn.multi) f += P;
    if (kn.pl) f += lanes * (kn.pl + 1);
    return sizeof(float) * f;
}

// One shape's kernel, lanes and LDS on a device of cus compute units and lds_max
// bytes of LDS (asked for once a choice, which tries up to forty shapes), or
// false if no instantiation holds it.
static bool gang_layout(int fitness, const SwarmArgs &a, int cus, int lds_max, int C, uint32_t P, GangShape *out)
{
    int nk = 0;
    const GangKernel *tab = gang_kernels(fitness, &nk);
    const uint32_t L = ((uint32_t)a.D + C - 1) / C;
    const uint64_t lanes = ((uint64_t)P * L + 63) / 64 * 64, G = ((uint64_t)a.N + P - 1) / P;
    if (G > GANG_PARTS_MAX || G > (uint64_t)cus) return false;
    if (P < 16) return false;
    for (int q = 0; q < nk; ++q) {
        const GangKernel &kn = tab[q];
        if (kn.C != C || kn.multi != (L > 1) || (kn.tail && L != 2) || lanes > (uint64_t)kn.max_lanes) continue;
        if (kn.uni != (P % 64 == 0)) continue;
        const size_t lds = gang_lds(fitness, a.D, kn, P, L);
        if (lds + sizeof(GangShared) + 1024 > (size_t)lds_max) continue;
        *out = GangShape{kn.fn, C, P, L, (uint32_t)G, (uint32_t)lanes, lds};
        return true;
    }
    return false;
}

// The shape: chunk C and particles P of a part.  An iteration's time is the
// lanes' C dimensions (45 to 60 vector instructions each, all wavefronts of a
// SIMD in turn), the fold of D - C staged terms (about 8 cycles each) and the
// meeting (0.9 us for few parts, 1.3 at 128, 2.2 at 256, and 0.5 more where
// the gbest changed).  Measured on Rastrigin alone over N = 32 .. 262144 and D = 1
// .. 300, us per iteration of the shape taken / the best of the others / the step
// launches or the one-workgroup run; the other functions take the same shapes,
// except where their settling matters (below):
//   one part (no meeting; one_part) while its lanes hold the swarm: N = 40, D =
//     20 1.8 / 2.1 / 2.1; 100, 12 1.85 / 2.6 / 2.24; 257, 5 1.92 / 2.2 / 2.2;
//     624, 2 1.66 / 1.94 / 1.66 (60 iterations; 0.89 / 0.81 / 1.26 of 300);
//     of very few deep particles the one-workgroup run is faster, which has
//     more lanes for each (100 iterations: Cubic N = 4, D = 130 455 / 336 us, Rastrigin
//     N = 8, D = 250 643 / 505, N = 4, D = 24 185 / 165; level at N = 32, D = 40)
//   D <= 2: 256 particles of a part, one lane each (C = 1 for D = 1): N =
//     16384, D = 2 1.05 / 1.08 / 6.27
//   D <= 4: pairs of lanes with few particles each, 32 of a part, below N =
//     6000 (2000, 3: 1.65 / 1.72 / 4.85), one lane beyond (8000, 4: 1.92 /
//     1.97 / 7.83)
//   D <= 16: C = 2 while the particles are few (N = 1000, D = 8: 2.80 / 3.1 /
//     5.34; 4000, 11: 3.20 / 3.34 / 12.8), C = 8 beyond (16384, 16: 4.03 /
//     4.2 / 13.2); D <= 8 keeps C = 2 up to 1024 lanes a part (32768, 5: 2.18
//     / 2.23 / 8.8)
//   larger D: C = 8, with 64 particles of a part up to D = 64 (N = 4000, D =
//     30: 3.86 / 4.1 / 12.3), and from 16 on beyond (1000, 128: 5.56 / 6.2 /
//     13.8), where folding dominates and more parts share it
//   parts: about 128 where the lanes allow it (N = 32768, D = 7: 4.26 at 128
//     parts, 4.3 at 256), up to 256 else (16384, 100: 7.1 at 256)
//   larger chunks where smaller ones need more lanes than a part has: N =
//     65536: D = 64 C = 16 10.1 / 15.1 (C = 64) / 23.3; D = 128 C = 64 19.9 /
//     39.2; N = 262144: D = 16 8.3 / 25.2, D = 30 C = 32 16.2 / 37.9
bool gang_shape(int fitness, const SwarmArgs &a, int64_t t0, int64_t T, GangShape *out)
{
    int cus = 0, lds_max = 0;
    if (!gang_device(&cus, &lds_max)) return false;
    auto layout = [&](int c, uint32_t P, GangShape *s) { return gang_layout(fitness, a, cus, lds_max, c, P, s); };
    if (const char *env = getenv("PSO_GANG_SHAPE")) { // "C,P": forced (tests, measurements)
        int c = 0, p = 0;
        return sscanf(env, "%d,%d", &c, &p) == 2 && c >= 1 && p >= 16 && p <= 1024 &&
               layout(c, (uint32_t)p, out);
    }
    const int D = a.D;
    const uint32_t N = a.N;
    if ((N < 32 && D > 24) || (N <= 16 && D > 16)) return false;
    // Where the gbest changes in most iterations, no block of them pays for what
    // surrounds it, and the one-workgroup run is faster (us of a run, here / there:
    // Sphere D = 2, T = 300: N = 641 445 / 331, 1024 475 / 375; N = 1500 T = 100
    // 223 / 185; Ackley N = 600, D = 2, T = 100 207 / 182, N = 800, D = 1 195 / 175);
    // at T = 600 the two are level, and Rastrigin and Cubic settle too early.
    // Iterations count from Step 1: a run that goes on from one before it has
    // settled (Sphere D = 2, N = 1000, 200 iterations more: 120 / 240).
    const bool late = settles_late(fitness);
    const int64_t end = t0 + T;
    if (late && D == 2 && N > 640 && N <= 1600 && end < (N <= 1300 ? 500 : 300)) return false;
    if (fitness == F_ACKLEY && D <= 2 && N > 384 && N <= 1024 && end < 200) return false;
    // A brief run stays in one part longer (settles_late; us of 200 iterations, one
    // part / more: Rosenbrock D = 3, N = 800 400 / 490; Rastrigin D = 2, N = 641
    // 203 / 196, of 100 137 / 146; Sphere D = 2, N = 641 of 600 621 / 697; Rosenbrock
    // D = 10, N = 343 of 300 818 / 919, D = 12, N = 500 864 / 950).
    const bool brief = end < 200, longer = late && end < 800;
    const uint32_t most2 = brief ? 1024 : longer && D == 2 ? 768 : 640, most4 = brief || longer ? 960 : 768;
    const uint32_t most8 = longer && D <= 12 ? 512 : 256;
    if (one_part(N, D, most2, most4, most8, [&](int c, uint32_t P) { return layout(c, P, out); })) return true;
    // Several parts: the state's way in and out of the registers and the
    // rendezvous of up to 256 parts have to pay.  Against the step launches (us of
    // a run of T, here / there): N = 4000, D = 30 T = 1 35 / 29, 2 39 / 39; N =
    // 131072: D = 2 T = 1 59 / 26, 4 65 / 49, 8 70 / 74; D = 16 T = 2 63 / 50, 4 66 /
    // 78; D = 30 T = 1 80 / 51, 2 84 / 92; N = 262144: D = 1 T = 4 90 / 56, 8 100 / 93;
    // D = 8 T = 4 102 / 79, 6 110 / 106; D = 30 T = 2 129 / 95, 4 155 / 165 (its runs of
    // eight and nine at D <= 4 are held, level with the steps: 93 / 92).  Up to
    // N = 65536 one iteration of D <= 16 is level with the steps.  Rastrigin and
    // Cubic improve fewer pbests early on, which the steps gain from (D = 43, T = 2 and
    // 3, of the steps' time: N = 36000 1.25 and 1.03, N = 97000 1.55 and 1.21; Sphere
    // 0.96 and 0.77, 0.67 and 0.54).
    const bool light = fitness == F_RASTRIGIN || fitness == F_CUBIC;
    const bool most = N > 131072;
    int64_t shortest = N <= 65536 ? (D > 16 ? 2 : 1) : D <= 4 ? (most ? 10 : 8) : D <= 16 ? (most ? 6 : 4) : (most ? 4 : 2);
    if (light && D > 16 && N > 24000) shortest = N > 65536 ? 5 : 4;
    if (T < shortest) return false;
    int c = D == 1 ? 1 : 2;
    uint32_t pmin = 256;
    if (D > 64) c = 8, pmin = 16;
    else if (D > 16) c = 8, pmin = 64;
    else if (D > 8) c = N < 6000 ? 2 : 8, pmin = N < 6000 ? 16 : 64;
    else if (D > 4) pmin = 16;
    else if (D > 2) c = N < 6000 ? 2 : 4, pmin = N < 6000 ? 32 : 256;
    for (; c <= 64; c *= 2) {
        const uint32_t L = ((uint32_t)D + c - 1) / c;
        uint32_t P = c >= 16 ? std::max(pmin, 64u) : pmin;
        if (L == 1) P = std::max(P, 64u);
        GangShape s;
        bool ok = layout(c, P, &s);
        // more particles of a part while there are too many parts
        while (P < 1024 && (a.N + P - 1) / P > (D <= 2 ? 256u : 128u)) {
            P *= 2;
            const bool more = layout(c, P, &s);
            if (ok && !more) break;
            ok = more;
        }
        if (ok) {
            *out = s;
            return true;
        }
    }
    return false;
}

hipError_t launch_gang(const SwarmArgs &a, const GangShape &s, uint32_t T, unsigned long long *words,
                       hipStream_t stream)
{
    int cus = 0, lds_max = 0;
    if (!gang_device(&cus, &lds_max)) return hipErrorInvalidDevice;
    // the most any swarm may ask for, so concurrent callers never lower it
    hipError_t e = hipFuncSetAttribute(s.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       lds_max - (int)sizeof(GangShared) - 1024);
    if (e != hipSuccess) return e;
    SwarmArgs args = a;
    GangArgs ga{};
    ga.T = T;
    ga.P = s.P;
    ga.L = s.L;
    ga.c1s = std::ldexp(a.c1, -24);
    ga.c2s = std::ldexp(a.c2, -24);
    ga.words = words;
    ga.block_ratio = block_ratio(s.C, s.L, s.lanes, s.G, 1.0f);
    void *params[] = {&args, &ga};
    return hipLaunchKernel(s.fn, dim3(s.G), dim3(s.lanes), params, s.lds, stream);
}

} // namespace pso
