// pso_hold.hip -- a run by one resident workgroup per compute unit that holds
// part of the state on the chip and streams the rest, for swarms whose state
// the resident gang cannot hold.
//
// The grid step moves the whole state through the memory-side cache in every
// iteration (809 MB at N = 2^20, D = 32, at 6.7 TB/s at the fabric; a large copy
// 5.4), and that bounds it: the vector instructions take half of that time.  256 compute units
// hold 128 MiB of registers and 40 MiB of LDS that live as long as a
// workgroup.  Here a part's 512 lanes each take 16-byte groups of particles
// (four binary32, two binary64); of a lane's first group, four or five
// pairs of dimensions stay in registers (24 registers a pair, of the 256 a lane
// has at two wavefronts per SIMD) and up to three more in LDS (48 KiB a pair), from
// the first iteration of a launch to the last.  The other dimensions, and a
// lane's further groups, are read and written as by the grid step.  Held and
// streamed pairs alternate, so that a streamed pair's loads are in flight while
// a held pair is computed.
//
// The parts meet once per iteration, as the resident gang's: a 64-byte line of
// tagged words each (fitness order bits, index), the winner's position in
// tagged words read only from it; relaxed device-scope atomics, bounded waits,
// and a rendezvous that leaves the state untouched where the parts are not all
// resident.  The arithmetic of every element is the grid step's, so the results
// are the same bits; the cosine, clamps and uniforms take the shorter forms
// that are exact where gang_accepts says so.
//
// Rastrigin, D = 32: N = 2^20, binary32, 200 iterations 24.3 -> 18.0 ms (bound
// by the three quarters of the state that still stream, 580 MB an iteration at
// 6.2 to 6.4 TB/s); N = 2^18, binary64, 50 iterations 4.1 -> 2.4 ms (the same, and
// by the double cosine).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "pso_f64_device.hpp"
#include "pso_gang_device.hpp"
#include "pso_hold.hpp"
#include "pso_quad.hpp"

namespace pso {

namespace {

constexpr int LANES = 512, LDS_PAIRS_MAX = 3;
// Pairs held in registers: five, or four beside the double cosine.  All forms
// spill, with five pairs 18 to 26 registers in binary32 and 8 to 14 in binary64,
// with four beside the cosine 20 and 31, and they are the fastest all the same:
// D = 32, ms, binary32 N = 2^20, 100 iterations, 3 / 4 / 5 / 6 pairs: Rastrigin 9.95 /
// 9.60 / 9.33 / 13.1, Sphere 10.0 / 9.73 / 9.48 / 9.61; binary64 N = 2^18, 50
// iterations, 3 / 4 / 5: Rastrigin 2.33 / 2.33 / 2.49, Ackley 2.34 / 2.33 / 2.57.  Two
// pairs in LDS instead of three: 9.61 and 2.41.
template <class T>
constexpr int held_of(int fitness)
{
    return sizeof(T) == 8 && (fitness == F_RASTRIGIN || fitness == F_ACKLEY) ? 4 : 5;
}
constexpr size_t LDS_PAIR_BYTES = (size_t)6 * 16 * LANES;

struct R32 {
    using T = float;
    typedef float V __attribute__((ext_vector_type(4)));
    using Args = SwarmArgs;
    static constexpr int VEC = 4, WORDS = 1; // particles of a group, words of a value
    template <int FIT>
    using Fit = Fitness<FIT>;
    template <int FIT>
    static __device__ __forceinline__ void add(Fitness<FIT> &f, float z, int d)
    {
        if constexpr (FIT == F_ROSENBROCK) {
            f.add(z, d);
        } else {
            f.acc = f.acc + gang_term<FIT>(z);
            if constexpr (FIT == F_ACKLEY) f.aux = f.aux + cos2pi_small(z);
        }
    }
    static __device__ __forceinline__ unsigned long long ord(float f) { return make_key(f, 0u) >> 32; }
    static __device__ __forceinline__ float clamp_v(float v, float m) { return clamp_sym(v, m); }
    static __device__ __forceinline__ float clamp_x(float v, float lo, float hi) { return clamp_pos(v, lo, hi); }
};

struct R64 {
    using T = double;
    typedef double V __attribute__((ext_vector_type(2)));
    using Args = Swarm64Args;
    static constexpr int VEC = 2, WORDS = 2;
    template <int FIT>
    using Fit = Fitness64<FIT>;
    template <int FIT>
    static __device__ __forceinline__ void add(Fitness64<FIT> &f, double z, int d) { f.add(z, d); }
    static __device__ __forceinline__ unsigned long long ord(double f) { return ord64(f); }
    static __device__ __forceinline__ double clamp_v(double v, double m) { return clamp_x(v, -m, m); }
    // equals the comparisons for finite v and bounds that are not -0
    static __device__ __forceinline__ double clamp_x(double v, double lo, double hi)
    {
        return __builtin_fmin(__builtin_fmax(v, lo), hi);
    }
};

template <class T>
struct HoldArgs {
    uint32_t T_, slots, groups;
    int lds_pairs;
    T c1s, c2s; // c1 2^-24, c2 2^-24 (exact)
    unsigned long long *words;
};

struct HoldShared {
    unsigned long long ord[2][LANES / 64]; // each wavefront's least candidate, rows alternating
    uint32_t idx[2][LANES / 64];
    unsigned long long win; // the meeting's result, ~0 if none
    uint32_t win_idx, err, go;
};

// A pair's x, v, p of one group.
template <class V>
struct Pair {
    V x[2], v[2], p[2];
};

template <bool KEEP, class V, class T>
__device__ __forceinline__ V load16(const T *at)
{
    if constexpr (KEEP) return *reinterpret_cast<const V *>(at);
    else return __builtin_nontemporal_load(reinterpret_cast<const V *>(at));
}

template <bool KEEP, class V, class T>
__device__ __forceinline__ void store16(T *at, V v)
{
    if constexpr (KEEP) *reinterpret_cast<V *>(at) = v;
    else __builtin_nontemporal_store(v, reinterpret_cast<V *>(at));
}

template <class V, int VEC>
__device__ __forceinline__ auto element(const V &v, uint32_t e)
{
    auto r = v[0];
#pragma unroll
    for (int q = 1; q < VEC; ++q) r = e == (uint32_t)q ? v[q] : r;
    return r;
}

// KEEP: the streamed rows fit the memory-side cache; else v and p stream past
// it and x has it for itself (Rastrigin D = 32, N = 2^20: 18.1 ms, with v kept
// too 18.2, with p as well 20.2).
template <class R, int FIT, bool KEEP>
__global__ void __launch_bounds__(LANES) __attribute__((amdgpu_waves_per_eu(2)))
k_hold(typename R::Args a, HoldArgs<typename R::T> h)
{
    using T = typename R::T;
    using V = typename R::V;
    using Fit = typename R::template Fit<FIT>;
    constexpr int VEC = R::VEC, WORDS = R::WORDS, HELD = held_of<T>(FIT);
    constexpr uint32_t ALL = (1u << VEC) - 1u;
    __shared__ HoldShared sh;
    extern __shared__ __attribute__((aligned(16))) char s_hold[]; // read in 16-byte vectors
    auto *c = a.ctrl;
    const int D = a.D, DP = (D + 1) / 2, M = h.lds_pairs;
    const uint32_t G = gridDim.x, part = blockIdx.x, tid = threadIdx.x, slots = h.slots;
    V *const s_pair = reinterpret_cast<V *>(s_hold) + tid; // [pair][x0 x1 v0 v1 p0 p1][lane]
    T *const s_g = reinterpret_cast<T *>(s_hold + (size_t)M * LDS_PAIR_BYTES), *const s_shift = s_g + 2 * DP;
    const uint32_t NV = (a.N + VEC - 1) / VEC, first = part * h.groups;
    const uint32_t count = first < NV ? (h.groups < NV - first ? h.groups : NV - first) : 0u;

    // control block, before any part can write it back
    unsigned long long gord;
    uint32_t gidx;
    if constexpr (VEC == 4) {
        gord = c->gkey_prev >> 32;
        gidx = (uint32_t)c->gkey_prev;
    } else {
        gord = c->gord;
        gidx = c->gidx;
    }
    long long giter = c->giter;
    const long long t0 = c->t;
    bool stop = c->stop != 0u;
    const T tol = c->tol, fstar = c->fstar;

    // this part's meeting words (both parities) to zero, then the rendezvous
    unsigned long long *const kw = h.words, *const pw = h.words + (size_t)2 * KEY_STRIDE * G;
    const uint32_t pstride = (uint32_t)(WORDS * D);
    for (uint32_t q = tid; q < 2 * (3 + pstride); q += LANES) {
        const uint32_t par = q & 1, w = q >> 1;
        unsigned long long *dst = w < 3 ? kw + ((size_t)par * G + part) * KEY_STRIDE + w
                                        : pw + ((size_t)par * G + part) * pstride + (w - 3);
        __hip_atomic_store(dst, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int d = (int)tid; d < 2 * DP; d += LANES) {
        s_g[d] = d < D ? a.gpos[d] : (T)0;
        s_shift[d] = d < D ? a.shift[d] : (T)0;
    }
    if (tid == 0) sh.err = 0;
    __syncthreads();
    if (tid == 0) {
        __threadfence(); // the zeroed words precede the arrival
        unsigned int *here;
        if constexpr (VEC == 4) here = reinterpret_cast<unsigned int *>(&c->gang_arrive);
        else here = &c->gang_here;
        if (atomicAdd(here, 1u) == G - 1) atomicCAS(&c->gang_state, 0u, GANG_GO);
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

    const uint32_t i0 = (first + tid) * VEC; // the lane's first group's particles
    const bool has0 = tid < count;
    uint32_t pend = 0; // per slot, VEC bits: the pbest position is x, its streamed dimensions not yet in p
    for (uint32_t s = 0; s < slots; ++s) {
        const uint32_t g = s * LANES + tid;
        if (g >= count) continue;
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            if (a.pend[(size_t)(first + g) * VEC + e]) pend |= 1u << (s * VEC + e);
    }
    Pair<V> H[HELD];
#pragma unroll
    for (int r = 0; r < HELD; ++r)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            H[r].x[q] = H[r].v[q] = H[r].p[q] = V(0);
            if (has0 && 4 * r + q < D) {
                const size_t at = (size_t)(4 * r + q) * a.Np + i0;
                H[r].x[q] = *reinterpret_cast<const V *>(a.x + at);
                H[r].v[q] = *reinterpret_cast<const V *>(a.v + at);
                H[r].p[q] = *reinterpret_cast<const V *>(a.p + at);
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    if (pend >> e & 1u) H[r].p[q][e] = H[r].x[q][e];
            }
        }
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int d = 2 * (2 * HELD + m) + q;
            if (!has0 || d >= D) continue;
            const size_t at = (size_t)d * a.Np + i0;
            const V x = *reinterpret_cast<const V *>(a.x + at);
            V p = *reinterpret_cast<const V *>(a.p + at);
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (pend >> e & 1u) p[e] = x[e];
            s_pair[(6 * m + q) * LANES] = x;
            s_pair[(6 * m + 2 + q) * LANES] = *reinterpret_cast<const V *>(a.v + at);
            s_pair[(6 * m + 4 + q) * LANES] = p;
        }

    // Eq. 1, Eq. 2 and the fitness terms of pair pr of the group at i
    auto update = [&](int pr, uint32_t i, uint32_t t, Pair<V> &S, Fit (&fit)[VEC]) __attribute__((always_inline)) {
        U4 u[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) u[e] = philox4x32_10(a.k0, a.k1, (uint32_t)pr, i + e, t, TAG_VEL);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int d = 2 * pr + q;
            if (d >= D) break;
            const T g = s_g[d], o = s_shift[d];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const T r1 = (T)(word_r1(u[e], q) >> 8), r2 = (T)(word_r2(u[e], q) >> 8);
                const T x = S.x[q][e];
                const T own = (a.w * S.v[q][e]) + ((h.c1s * r1) * (S.p[q][e] - x));
                const T nv = R::clamp_v(own + ((h.c2s * r2) * (g - x)), a.vmax);
                const T xn = R::clamp_x(x + nv, a.lo, a.hi);
                S.v[q][e] = nv;
                S.x[q][e] = xn;
                R::template add<FIT>(fit[e], xn - o, d);
            }
        }
    };
    auto fetch = [&](int pr, uint32_t i, Pair<V> &S) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (2 * pr + q >= D) break;
            const size_t at = (size_t)(2 * pr + q) * a.Np + i;
            S.x[q] = load16<true, V>(a.x + at);
            S.v[q] = load16<KEEP, V>(a.v + at);
            S.p[q] = load16<KEEP, V>(a.p + at);
        }
    };
    // a streamed pair: marked particles' pbest position is the x just read
    auto streamed = [&](int pr, uint32_t i, uint32_t t, uint32_t marks, bool line, Pair<V> &S, Fit (&fit)[VEC]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (marks >> e & 1u) S.p[q][e] = S.x[q][e];
        update(pr, i, t, S, fit);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (2 * pr + q >= D) break;
            const size_t at = (size_t)(2 * pr + q) * a.Np + i;
            store16<true, V>(a.x + at, S.x[q]);
            store16<KEEP, V>(a.v + at, S.v[q]);
            if (line) store16<KEEP, V>(a.p + at, S.p[q]);
        }
    };

    // Every second wavefront takes its groups in the opposite order: some stream
    // while others compute held pairs.  The first streamed pair of an iteration
    // is read ahead of the meeting.
    const bool turned = (__builtin_amdgcn_readfirstlane((int)(tid >> 6)) & 1) != 0;
    const uint32_t s_first = turned ? slots - 1 : 0u;
    const bool on_first = s_first * LANES + tid < count;
    Pair<V> B;
    auto fetch_first = [&]() __attribute__((always_inline)) {
        const int pr = s_first == 0 ? 1 : 0;
        if (on_first && pr < DP) fetch(pr, (first + s_first * LANES + tid) * VEC, B);
    };
    fetch_first();
    uint32_t n_imp = 0, done = 0;
    while (done < h.T_ && !stop) {
        const uint32_t t = (uint32_t)(t0 + done + 1), seq = done + 1, par = seq & 1;
        unsigned long long my_k = ~0ull;
        uint32_t my_i = NO_IDX;
        for (uint32_t n = 0; n < slots; ++n) {
            const uint32_t s = turned ? slots - 1 - n : n;
            const uint32_t g = s * LANES + tid;
            const bool on = g < count;
            const uint32_t marks = pend >> (s * VEC) & ALL;
            // p is written by whole 64-byte lines that hold a mark
            const bool line = ((__ballot(on && marks != 0u) >> ((tid & 63u) & ~3u)) & 0xFull) != 0;
            if (!on) continue;
            const uint32_t i = (first + g) * VEC;
            const V pf_old = *reinterpret_cast<const V *>(a.pf + i);
            Fit fit[VEC];
            int pr = 0;
            if (s == 0) {
#pragma unroll
                for (int r = 0; r < HELD; ++r) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (2 * r + 1 < DP && (r > 0 || n > 0)) fetch(2 * r + 1, i, B);
                    if (2 * r < DP) update(2 * r, i, t, H[r], fit);
                    if (2 * r + 1 < DP) streamed(2 * r + 1, i, t, marks, line, B, fit);
                }
                pr = 2 * HELD + M;
                if (pr < DP) fetch(pr, i, B);
                for (int m = 0; m < M; ++m) {
                    Pair<V> S;
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        S.x[q] = s_pair[(6 * m + q) * LANES];
                        S.v[q] = s_pair[(6 * m + 2 + q) * LANES];
                        S.p[q] = s_pair[(6 * m + 4 + q) * LANES];
                    }
                    update(2 * HELD + m, i, t, S, fit);
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        s_pair[(6 * m + q) * LANES] = S.x[q];
                        s_pair[(6 * m + 2 + q) * LANES] = S.v[q];
                    }
                }
            } else if (n > 0) {
                fetch(0, i, B);
            }
            for (; pr < DP; ++pr) {
                Pair<V> S = B;
                if (pr + 1 < DP) fetch(pr + 1, i, B);
                streamed(pr, i, t, marks, line, S, fit);
            }
            // Step 4 (strict; NaN never improves) and the candidates
            uint32_t marks_new = 0;
            V pf_new = pf_old;
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                if (i + e >= a.N) continue;
                const T f = fit[e].value(D);
                if (!(f < pf_old[e])) continue;
                pf_new[e] = f;
                marks_new |= 1u << e;
                const unsigned long long o = R::ord(f);
                if (o < gord || (o == gord && i + e < gidx)) lexmin(my_k, my_i, o, i + e);
            }
            pend = (pend & ~(ALL << (s * VEC))) | marks_new << (s * VEC);
            if (marks_new) {
                *reinterpret_cast<V *>(a.pf + i) = pf_new;
                n_imp += (uint32_t)__popc(marks_new);
            }
            if (s == 0 && marks_new) {
#pragma unroll
                for (int r = 0; r < HELD; ++r)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
#pragma unroll
                        for (int e = 0; e < VEC; ++e)
                            if (marks_new >> e & 1u) H[r].p[q][e] = H[r].x[q][e];
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const V x = s_pair[(6 * m + q) * LANES];
                        V p = s_pair[(6 * m + 4 + q) * LANES];
#pragma unroll
                        for (int e = 0; e < VEC; ++e)
                            if (marks_new >> e & 1u) p[e] = x[e];
                        s_pair[(6 * m + 4 + q) * LANES] = p;
                    }
            }
        }
        // Step 5: the part's candidate
        unsigned long long wk = my_k;
        uint32_t wi = my_i;
        wave_lexmin_sparse(wk, wi);
        if ((tid & 63u) == 0) {
            sh.ord[par][tid >> 6] = wk;
            sh.idx[par][tid >> 6] = wi;
        }
        __syncthreads(); // and this iteration's stores are visible to the workgroup
        wk = ~0ull;
        wi = NO_IDX;
#pragma unroll
        for (int q = 0; q < LANES / 64; ++q) lexmin(wk, wi, sh.ord[par][q], sh.idx[par][q]);
        const unsigned long long ptag = (unsigned long long)seq << 32;
        unsigned long long *const line_w = kw + ((size_t)par * G + part) * KEY_STRIDE;
        if (wi != NO_IDX) {
            unsigned long long *dst = pw + ((size_t)par * G + part) * pstride;
            auto post = [&](int d, T value) __attribute__((always_inline)) {
                unsigned long long bits = 0;
                __builtin_memcpy(&bits, &value, sizeof value);
#pragma unroll
                for (int q = 0; q < WORDS; ++q)
                    __hip_atomic_store(&dst[WORDS * d + q], ptag | (uint32_t)(bits >> (32 * q)), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            };
            const uint32_t e = wi % VEC;
            const bool held = wi / VEC - first < (uint32_t)LANES; // a first group: some dimensions are on the chip
            if (held && my_i == wi) {
#pragma unroll
                for (int r = 0; r < HELD; ++r)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        if (4 * r + q < D) post(4 * r + q, element<V, VEC>(H[r].x[q], e));
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const int d = 2 * (2 * HELD + m) + q;
                        if (d < D) post(d, element<V, VEC>(s_pair[(6 * m + q) * LANES], e));
                    }
            }
            if (tid < 64) {
                for (int d = (int)tid; d < D; d += 64) {
                    const int pr = d >> 1;
                    if (held && (pr < 2 * HELD ? (pr & 1) == 0 : pr < 2 * HELD + M)) continue;
                    post(d, a.x[(size_t)d * a.Np + wi]);
                }
            }
        }
        if (tid < 3)
            __hip_atomic_store(line_w + tid, ptag | (tid == 0 ? (uint32_t)(wk >> 32) : tid == 1 ? (uint32_t)wk : wi),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (done + 1 < h.T_) fetch_first();
        // the meeting
        if (tid < 64) {
            const unsigned long long w0 = wall_clock64();
            unsigned long long bk = ~0ull;
            uint32_t bi = NO_IDX, bp = 0;
            for (uint32_t b = tid; b < G; b += 64) {
                const unsigned long long *src = kw + ((size_t)par * G + b) * KEY_STRIDE;
                unsigned long long v0, v1, v2;
                for (uint32_t spins = 0;;) {
                    v0 = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    v1 = __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    v2 = __hip_atomic_load(src + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((v0 >> 32) == seq && (v1 >> 32) == seq && (v2 >> 32) == seq) break;
                    if ((++spins & 63u) == 0u && wall_clock64() - w0 > GANG_TICKS) {
                        sh.err = 1u;
                        break;
                    }
                }
                const unsigned long long k = v0 << 32 | (uint32_t)v1;
                const uint32_t ki = (uint32_t)v2;
                if (ki != NO_IDX && (k < bk || (k == bk && ki < bi))) {
                    bk = k;
                    bi = ki;
                }
            }
            wave_lexmin_sparse(bk, bi);
            if (bi != NO_IDX) { // uniform
                bp = bi / VEC / h.groups;
                const unsigned long long *src = pw + ((size_t)par * G + bp) * pstride;
                for (uint32_t d = tid; d < (uint32_t)D; d += 64) {
                    unsigned long long bits = 0;
#pragma unroll
                    for (int q = 0; q < WORDS; ++q) {
                        unsigned long long w;
                        for (uint32_t spins = 0;;) {
                            w = __hip_atomic_load(&src[WORDS * d + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            if ((w >> 32) == seq) break;
                            if ((++spins & 63u) == 0u && wall_clock64() - w0 > GANG_TICKS) {
                                sh.err = 1u;
                                break;
                            }
                        }
                        bits |= (w & 0xFFFFFFFFull) << (32 * q);
                    }
                    T value;
                    __builtin_memcpy(&value, &bits, sizeof value);
                    s_g[d] = value;
                }
            }
            if (tid == 0) {
                sh.win = bk;
                sh.win_idx = bi;
            }
        }
        __syncthreads();
        if (sh.err) break; // uniform; the state is lost and the caller told
        ++done;
        const uint32_t win_idx = sh.win_idx;
        if (win_idx != NO_IDX) {
            gord = sh.win;
            gidx = win_idx;
            giter = t0 + done;
        }
        T gbest;
        if constexpr (VEC == 4) {
            const unsigned long long gkey = gord << 32 | gidx;
            if (part == 0 && tid == 0 && a.hist) a.hist[t & (HIST_CAP - 1)] = gkey;
            gbest = key_fitness(gkey);
        } else {
            gbest = ord64_value(gord);
        }
        stop = tol > (T)0 && __builtin_fabs(gbest - fstar) < tol;
    }

#pragma unroll
    for (int r = 0; r < HELD; ++r)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (!has0 || 4 * r + q >= D) continue;
            const size_t at = (size_t)(4 * r + q) * a.Np + i0;
            *reinterpret_cast<V *>(a.x + at) = H[r].x[q];
            *reinterpret_cast<V *>(a.v + at) = H[r].v[q];
            *reinterpret_cast<V *>(a.p + at) = H[r].p[q];
        }
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int d = 2 * (2 * HELD + m) + q;
            if (!has0 || d >= D) continue;
            const size_t at = (size_t)d * a.Np + i0;
            *reinterpret_cast<V *>(a.x + at) = s_pair[(6 * m + q) * LANES];
            *reinterpret_cast<V *>(a.v + at) = s_pair[(6 * m + 2 + q) * LANES];
            *reinterpret_cast<V *>(a.p + at) = s_pair[(6 * m + 4 + q) * LANES];
        }
    for (uint32_t s = 0; s < slots; ++s) {
        const uint32_t g = s * LANES + tid;
        if (g >= count) continue;
#pragma unroll
        for (int e = 0; e < VEC; ++e) a.pend[(size_t)(first + g) * VEC + e] = (uint8_t)(pend >> (s * VEC + e) & 1u);
    }
    if constexpr (VEC == 4) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) n_imp += __shfl_xor(n_imp, off, 64);
        if ((tid & 63u) == 0 && n_imp) atomicAdd(&c->improved, (unsigned long long)n_imp);
        if (tid == 0 && sh.err) atomicOr(&c->err, ERR_GANG_WAIT);
    } else {
        if (tid == 0 && sh.err) atomicOr(&c->err, 1u);
    }
    if (part != 0) return;
    for (int d = (int)tid; d < D; d += LANES) a.gpos[d] = s_g[d];
    if (tid == 0) {
        if constexpr (VEC == 4) {
            const unsigned long long gkey = gord << 32 | gidx;
            c->gkey = gkey;
            c->gkey_prev = gkey;
            c->pubkey = gkey;
        } else {
            c->gord = gord;
            c->gidx = gidx;
        }
        c->giter = giter;
        c->t = t0 + done;
        c->stop = stop ? 1u : 0u;
    }
}

template <class R, int FIT>
const void *hold_fn(bool keep)
{
    return keep ? reinterpret_cast<const void *>(k_hold<R, FIT, true>) : reinterpret_cast<const void *>(k_hold<R, FIT, false>);
}

template <class R>
bool shape_of(int fitness, const typename R::Args &a, int64_t T, HoldShape *out)
{
    const char *env = getenv("PSO_HOLD");
    if (env && !strcmp(env, "0")) return false;
    int cus = 0, lds_max = 0;
    if (fitness < F_SPHERE || fitness > F_CUBIC || a.D > GANG64_MAX_D_ALL || !gang_device(&cus, &lds_max)) return false;
    if (a.N < 16 * GANG_PARTS_MAX) return false; // gang64_words has every part's words from here on
    HoldShape s{};
    s.G = (uint32_t)std::min<int>(cus, (int)GANG_PARTS_MAX);
    const uint32_t NV = (a.N + R::VEC - 1) / R::VEC, DP = ((uint32_t)a.D + 1) / 2;
    s.groups = (NV + s.G - 1) / s.G;
    s.slots = (s.groups + LANES - 1) / LANES;
    if (s.slots * R::VEC > 32) return false; // the marks' bits
    const size_t head = sizeof(typename R::T) * 4 * DP + sizeof(HoldShared) + 1024;
    const uint32_t HELD = held_of<typename R::T>(fitness);
    s.lds_pairs = DP > 2 * HELD ? std::min<uint32_t>(DP - 2 * HELD, LDS_PAIRS_MAX) : 0u;
    while (s.lds_pairs > 0 && s.lds_pairs * LDS_PAIR_BYTES + head > (size_t)lds_max) --s.lds_pairs;
    s.lds = s.lds_pairs * LDS_PAIR_BYTES + sizeof(typename R::T) * 4 * DP;
    const uint32_t held = std::min<uint32_t>(HELD, (DP + 1) / 2) + s.lds_pairs;
    const double share = double(held) / (double(DP) * s.slots); // of the pairs, those held
    // Against the grid step (us per iteration, here / there):
    //  - Lanes: a part whose lanes mostly hold nothing streams with too few of
    //    them (Rastrigin D = 128: N = 2^18, half of the lanes, 116 / 169; 2^17,
    //    a quarter, 91 / 68).
    //  - Iterations: the held state is read and written once more than it would
    //    be, and the parts' rendezvous costs 10 to 15 us.  Binary32, N = 2^20,
    //    D = 4: 68 / 53 in a run of 2, 28 / 33 of 10, 17 / 27 of 100; binary64,
    //    N = 2^18, D = 32: 151 / 159 of 2, 48 / 79 of 100.
    //  - Share, binary32: N = 2^20, D = 32, a quarter held, 94 / 125; N = 1.5e6,
    //    D = 32, a sixth, 172 / 177; N = 3e6, D = 12, a twelfth, 142 / 137.  The
    //    binary64 grid steps are slower by more (N = 2^20, D = 16, an eighth, 114
    //    / 251; N = 2^22, D = 4, a sixteenth, 140 / 591).
    const bool wide = sizeof(typename R::T) == 8;
    if (!env && (s.groups < LANES / 2 || T < (wide ? 3 : 8) || (!wide && share < 0.1))) return false;
    const bool keep = 3.0 * sizeof(typename R::T) * double(a.Np) * a.D * (1.0 - share) <= 248.0 * 1048576;
    switch (fitness) {
    case F_SPHERE: s.fn = hold_fn<R, F_SPHERE>(keep); break;
    case F_RASTRIGIN: s.fn = hold_fn<R, F_RASTRIGIN>(keep); break;
    case F_ROSENBROCK: s.fn = hold_fn<R, F_ROSENBROCK>(keep); break;
    case F_ACKLEY: s.fn = hold_fn<R, F_ACKLEY>(keep); break;
    default: s.fn = hold_fn<R, F_CUBIC>(keep); break;
    }
    *out = s;
    return true;
}

template <class R>
hipError_t launch(const typename R::Args &a, const HoldShape &s, uint32_t T, unsigned long long *words, hipStream_t stream)
{
    int cus = 0, lds_max = 0;
    if (!gang_device(&cus, &lds_max)) return hipErrorInvalidDevice;
    // the most any swarm may ask for, so concurrent callers never lower it
    hipError_t e = hipFuncSetAttribute(s.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       lds_max - (int)sizeof(HoldShared) - 1024);
    if (e != hipSuccess) return e;
    typename R::Args args = a;
    HoldArgs<typename R::T> h{};
    h.T_ = T;
    h.slots = s.slots;
    h.groups = s.groups;
    h.lds_pairs = (int)s.lds_pairs;
    h.c1s = std::ldexp(a.c1, -24);
    h.c2s = std::ldexp(a.c2, -24);
    h.words = words;
    void *params[] = {&args, &h};
    return hipLaunchKernel(s.fn, dim3(s.G), dim3(LANES), params, s.lds, stream);
}

} // namespace

bool hold_shape(int fitness, const SwarmArgs &a, int64_t T, HoldShape *out) { return shape_of<R32>(fitness, a, T, out); }
bool hold_shape(int fitness, const Swarm64Args &a, int64_t T, HoldShape *out)
{
    return a.gang_words && shape_of<R64>(fitness, a, T, out);
}

size_t hold_words(int D) { return (size_t)2 * GANG_PARTS_MAX * (KEY_STRIDE + (size_t)D); }

hipError_t launch_hold(const SwarmArgs &a, const HoldShape &s, uint32_t T, unsigned long long *words, hipStream_t stream)
{
    return launch<R32>(a, s, T, words, stream);
}

hipError_t launch_hold(const Swarm64Args &a, const HoldShape &s, uint32_t T, hipStream_t stream)
{
    return launch<R64>(a, s, T, a.gang_words, stream);
}

} // namespace pso
