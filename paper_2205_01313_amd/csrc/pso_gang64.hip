// pso_gang64.hip -- the resident gang in binary64: pso_gang.hip's layout,
// meeting and blocks of iterations (described there) for the binary64 swarm.
//
// What differs: a lane's chunk takes twice the registers, so chunks are half
// as long; the key of a candidate -- order bits and index -- no longer fits
// one word, so a part's candidate is posted as three words of its line (the
// meeting's number, iteration and high half; low half; index), of which a
// reader needs the first alone where there is no candidate, and a part takes
// its minimum over its wavefronts lexicographically (wave_lexmin_sparse).
// Velocities and positions are finite (binary32 parameters cannot overflow a
// double), so the clamps are one maximum and one minimum; c1 2^-24 and c2 2^-24
// are exact.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "pso_f64.hpp"
#include "pso_f64_device.hpp"
#include "pso_gang.hpp"

namespace pso {

template <int FIT>
__device__ __forceinline__ double gang_term64(double z)
{
    if constexpr (FIT == F_RASTRIGIN) return z * z - 10.0 * cospi64(2.0 * z);
    else if constexpr (FIT == F_CUBIC) return z * z * z - 0.8 * z * z - 1000.0 * z + 8000.0;
    else return z * z; // Sphere, Ackley's first word
}

__device__ __forceinline__ double rosen_term64(double z, double zp)
{
    const double a = z - zp * zp;
    const double b = 1.0 - zp;
    return 100.0 * a * a + b * b;
}

// Equals the comparisons for finite v and bounds that are not -0
// (gang64_accepts).
__device__ __forceinline__ double clamp64(double v, double lo, double hi)
{
    return __builtin_fmin(__builtin_fmax(v, lo), hi);
}

template <int C, int PL>
struct LaneState64 {
    double x[C], v[C], p[C > PL ? C - PL : 1];
    double pf; // pbest fitness (chunk-0 lanes; -inf where there is no particle)
};

template <int C>
struct OwnHalf64 {
    double own[C], soc[C];
};

template <int C>
__device__ __forceinline__ void own_half64(const Swarm64Args &a, const Gang64Args &ga, int D, int d0, uint32_t i,
                                           uint32_t t, const LaneState64<C, 0> &S, OwnHalf64<C> &O)
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
                const double r1 = (double)((h ? u.c : u.a) >> 8), r2 = (double)((h ? u.d : u.b) >> 8);
                O.own[c + h] = (a.w * S.v[c + h]) + ((ga.c1s * r1) * (S.p[c + h] - S.x[c + h]));
                O.soc[c + h] = ga.c2s * r2;
            }
        }
    }
}

struct Gang64Shared {
    unsigned long long ord[2][16]; // each wavefront's least candidate, rows alternating
    uint32_t loc[2][16], ran[2][16];
    unsigned long long win_hi; // the meeting's result: iteration and high half, ~0 if none
    uint32_t win_lo, win_idx;
    uint32_t err, go;
};

// PL: dimensions of p kept in LDS, the last of the chunk (x, v and p of 32
// dimensions are 192 registers of the 256 a lane has at 512 lanes).
template <int FIT, int C, bool MULTI, bool UNI, bool SPEC, int MAXT, int PL = 0>
__global__ void __launch_bounds__(MAXT) k_gang64_resident(Swarm64Args a, Gang64Args ga)
{
    constexpr int W = FIT == F_ACKLEY ? 2 : 1;
    constexpr int Q = group_of(C), PR = C - PL;
    static_assert((C == 1 && !MULTI) || C % 2 == 0, "chunks hold whole Philox pairs");
    __shared__ Gang64Shared sh;
    // gbest position (two of them: a repeated block still reads the old one)
    // and shift (L * C floats each), then with MULTI the staged terms of the
    // chunks after the first -- a lane's are CP floats apart, word after word,
    // C + 1 of them so that consecutive lanes start on different banks and
    // every address is one register plus a constant --, each chunk's last z
    // (Rosenbrock), the improvement flags, and p's PL dimensions of each lane
    extern __shared__ double s_gang64[];
    Ctrl64 *c = a.ctrl;
    const int D = a.D;
    const uint32_t P = ga.P, G = gridDim.x, part = blockIdx.x, tid = threadIdx.x, T = blockDim.x;
    const int L = (int)ga.L, DL = L * C;
    double *s_gpos = s_gang64, *s_shift = s_gang64 + 2 * DL;
    constexpr int CP = C + 1, CW = W * CP;
    double *s_t = s_shift + DL, *s_last = s_t + (MULTI ? (size_t)CW * (L - 1) * P : 0);
    uint32_t *s_imp = reinterpret_cast<uint32_t *>(s_last + (FIT == F_ROSENBROCK ? (size_t)(L - 1) * P : 0));
    double *my_p = reinterpret_cast<double *>(s_imp + (MULTI ? P : 0)) + tid * (PL + 1); // odd stride: no bank conflicts
    int k_lane = MULTI ? (int)(tid / P) : 0;
    if (UNI) k_lane = __builtin_amdgcn_readfirstlane(k_lane);
    const int k = k_lane;
    const uint32_t j = MULTI ? tid - (uint32_t)k * P : tid;
    const int d0 = k * C;
    const uint32_t base = part * P, i = base + j;
    const bool valid = j < P && k < L && i < a.N;
    const bool folder = valid && k == 0;

    // control block, before any part can write it back
    unsigned long long gord = c->gord;
    uint32_t gidx = c->gidx;
    long long giter = c->giter;
    const long long t0 = c->t;
    bool stop = c->stop != 0u;
    const double tol = c->tol, fstar = c->fstar;

    // this part's meeting words (both parities) to zero, then the rendezvous
    unsigned long long *const kw = ga.words, *const pw = ga.words + (size_t)2 * KEY_STRIDE * G;
    const uint32_t pstride = 2 * (uint32_t)D;
    if (G > 1) {
        for (uint32_t q = tid; q < 2 * (3 + pstride); q += T) {
            const uint32_t par = q & 1, w = q >> 1;
            unsigned long long *dst = w < 3 ? kw + ((size_t)par * G + part) * KEY_STRIDE + w
                                            : pw + ((size_t)par * G + part) * pstride + (w - 3);
            __hip_atomic_store(dst, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    for (int d = (int)tid; d < DL; d += (int)T) {
        s_gpos[d] = d < D ? a.gpos[d] : 0.0;
        s_shift[d] = d < D ? a.shift[d] : 0.0;
    }
    if (tid == 0) sh.err = 0;
    __syncthreads();
    if (G > 1) {
        if (tid == 0) {
            __threadfence(); // the zeroed words precede the arrival
            if (atomicAdd(&c->gang_here, 1u) == G - 1) atomicCAS(&c->gang_state, 0u, GANG_GO);
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

    LaneState64<C, PL> S;
    S.pf = -__builtin_inf();
    {
        const bool pend = valid && a.pend[i] != 0;
#pragma unroll
        for (int e = 0; e < C; ++e) {
            double pe = 0.0;
            S.x[e] = S.v[e] = 0.0;
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

    double *s_g = s_gpos, *s_gn = s_gpos + DL; // in use, and the next one
    constexpr bool AHEAD = C <= 8; // room for the next iteration's own half in registers
    OwnHalf64<AHEAD ? C : 1> O;
    bool have_own = false;

    // a wavefront's least candidate (order bits, particle of the part) with
    // the iteration it stopped at, for the part's minimum
    auto leave = [&](int row, uint32_t ran, bool cand, unsigned long long ord) {
        unsigned long long kk = cand ? ord : ~0ull;
        uint32_t ii = cand ? j : NO_IDX;
        wave_lexmin_sparse(kk, ii);
        if ((tid & 63) == 0) {
            sh.ord[row][tid >> 6] = kk;
            sh.loc[row][tid >> 6] = ii;
            sh.ran[row][tid >> 6] = ran;
        }
    };
    // the part's: the earliest iteration, there the least (order bits, index)
    auto collect = [&](int row, uint32_t &ran, unsigned long long &kk, uint32_t &ii) {
        const uint32_t lane = tid & 63;
        kk = lane < T / 64 ? sh.ord[row][lane] : ~0ull;
        ii = lane < T / 64 ? sh.loc[row][lane] : NO_IDX;
        if (!__any(ii != NO_IDX)) return;
        ran = ii != NO_IDX ? sh.ran[row][lane] : ~0u;
        uint32_t first = ran;
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) first = min(first, (uint32_t)__shfl_xor((int)first, off, 64));
        first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first); // T / 64 <= 16 wavefronts
        if (ran != first) {
            kk = ~0ull;
            ii = NO_IDX;
        }
        wave_lexmin_sparse(kk, ii);
        ran = first;
    };

    // Steps 2-4 of iteration t; cand: this lane's particle improved and beats
    // the gbest, with fitness order bits ord.  With MULTI the wavefronts leave
    // their minima in row `row` before the last barrier.
    auto iterate = [&](uint32_t t, int row, bool &cand, unsigned long long &ord) {
        // opaque copies: the tests on them are scalar compares here, instead of
        // masks computed once before the loop and spilled
        int D = a.D, k = k_lane;
        asm volatile("" : "+s"(D));
        if constexpr (UNI) asm volatile("" : "+s"(k));
        const int d0 = k * C;
        Fitness64<FIT> fit;
        double zp = 0.0; // previous dimension's z (Rosenbrock)
        double *my_t = s_t + (MULTI && k > 0 ? (tid - P) * CW : 0u);
        if constexpr (AHEAD) {
            if (!have_own) own_half64<C>(a, ga, D, d0, i, t, S, O);
            have_own = false;
        }
#pragma unroll
        for (int e = 0; e < C; e += Q) {
            // large chunks: no scheduling across groups (their loads and draws
            // in flight together would not fit the registers)
            if constexpr (!AHEAD) __builtin_amdgcn_sched_barrier(0);
            if (d0 + e >= D) continue;
            double w0[Q], w1[W == 2 ? Q : 1];
#pragma unroll
            for (int q = e; q < e + Q; q += 2) {
                U4 u{};
                if constexpr (!AHEAD) u = philox4x32_10(a.k0, a.k1, (uint32_t)(d0 + q) >> 1, i, t, TAG_VEL);
#pragma unroll
                for (int h = 0; h < (C == 1 ? 1 : 2); ++h) {
                    const int c = q + h, d = d0 + c;
                    double own, soc;
                    if constexpr (AHEAD) {
                        own = O.own[c];
                        soc = O.soc[c];
                    } else {
                        const double r1 = (double)((h ? u.c : u.a) >> 8), r2 = (double)((h ? u.d : u.b) >> 8);
                        const double pc = c < PR ? S.p[c < PR ? c : 0] : my_p[c - PR];
                        own = (a.w * S.v[c]) + ((ga.c1s * r1) * (pc - S.x[c]));
                        soc = ga.c2s * r2;
                    }
                    const double nv = clamp64(own + (soc * (s_g[d] - S.x[c])), -a.vmax, a.vmax);
                    const double xn = clamp64(S.x[c] + nv, a.lo, a.hi);
                    S.v[c] = nv;
                    S.x[c] = xn;
                    const double z = xn - s_shift[d];
                    if constexpr (FIT == F_ROSENBROCK) {
                        // a chunk's first term needs the previous chunk's z
                        w0[c - e] = c == 0 ? z : rosen_term64(z, zp);
                    } else {
                        w0[c - e] = gang_term64<FIT>(z);
                        if constexpr (W == 2) w1[c - e] = cospi64(2.0 * z);
                    }
                    zp = z;
                }
            }
            if (MULTI && k > 0) {
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
        if constexpr (MULTI) {
            __syncthreads();
            if (folder) {
                // a batch of terms is loaded before they are added, so the sum
                // waits on LDS once a batch; terms past D are loaded (their
                // place exists) but not added
                constexpr int MOST = (MAXT <= 512 ? 16 : 8) / W; // terms of a batch
                constexpr int BS = C < MOST ? C : MOST, NB = MOST / BS; // of a chunk, chunks
                for (int kk = 1; kk < L; kk += NB) {
                    const double *r = s_t + ((uint32_t)(kk - 1) * P + j) * CW;
#pragma unroll
                    for (int q0 = 0; q0 < C; q0 += BS) {
                        double b0[NB][BS], b1[NB][W == 2 ? BS : 1], last[NB];
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
                            if (FIT == F_ROSENBROCK && q0 == 0) b0[n][0] = rosen_term64(b0[n][0], last[n]);
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
        ord = ~0ull;
        if (!MULTI || k == 0) {
            const double f = fit.value(D);
            imp = f < S.pf;
            if (imp) {
                S.pf = f;
                ord = ord64(f);
                cand = ord < gord || (ord == gord && i < gidx);
            }
        }
        if constexpr (MULTI) {
            if (k == 0 && j < P) s_imp[j] = imp ? 1u : 0u;
            leave(row, 0u, cand, ord);
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
    int K = 1, row = 0;
    float mean = 1.0f, since = 0.0f; // iterations between gbest changes, and since the last
    uint32_t seq = 0;
    stop = stop || (tol > 0.0 && fabs(ord64_value(gord) - fstar) < tol);
    while (done < (long long)ga.T && !stop) {
        ++seq;
        const uint32_t tb = (uint32_t)(t0 + done);
        const int n = SPEC ? (int)min((long long)K, (long long)ga.T - done) : 1;
        LaneState64<SPEC ? C : 1, PL> B;
        if constexpr (SPEC) {
            if (n > 1) B = S;
        }
        // the block: up to n iterations, as far as this wavefront's (part's)
        // first candidate
        uint32_t ran = 0, jw = 0, loc;
        bool cand = false;
        unsigned long long ord, kk;
        if constexpr (MULTI) {
            do {
                ++ran;
                row ^= 1;
                iterate(tb + ran, row, cand, ord); // ends with a barrier
                collect(row, jw, kk, loc);
            } while (ran < (uint32_t)n && loc == NO_IDX);
            jw = ran;
        } else {
            bool any;
            do {
                ++ran;
                iterate(tb + ran, row, cand, ord);
                any = __any(cand);
            } while (ran < (uint32_t)n && !any);
            // rows alternate: a row's last readers passed the barrier of the
            // block before this one
            row ^= 1;
            leave(row, ran, cand, ord);
            __syncthreads();
            collect(row, jw, kk, loc);
        }
        bool changed = loc != NO_IDX;
        uint32_t nc = jw; // iteration of the change within the block
        if (G > 1) {
            const uint32_t par = seq & 1, want = seq & 0xFFFFFFu;
            const unsigned long long ptag = (unsigned long long)seq << 32;
            unsigned long long *const line = kw + ((size_t)par * G + part) * KEY_STRIDE;
            if (changed && valid && j == loc) {
                unsigned long long *dst = pw + ((size_t)par * G + part) * pstride;
#pragma unroll
                for (int q = 0; q < C; ++q)
                    if (d0 + q < D) {
                        const unsigned long long bits = (unsigned long long)__double_as_longlong(S.x[q]);
                        __hip_atomic_store(&dst[2 * (d0 + q)], ptag | (uint32_t)bits, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                        __hip_atomic_store(&dst[2 * (d0 + q) + 1], ptag | (bits >> 32), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    }
            }
            if (tid == 0) {
                const unsigned long long hi = changed ? ((unsigned long long)jw << 32) | (kk >> 32) : 0xFFFFFFFFFFull;
                __hip_atomic_store(line, ((unsigned long long)want << 40) | hi, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                if (changed) {
                    __hip_atomic_store(line + 1, ptag | (uint32_t)kk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(line + 2, ptag | (base + loc), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if constexpr (AHEAD) {
                // meanwhile the next iteration's own half (of a block that
                // cannot be rolled back)
                if (n == 1 && done + 1 < (long long)ga.T) {
                    own_half64<C>(a, ga, D, d0, i, tb + 2, S, O);
                    have_own = true;
                }
            }
            if (tid < 64) {
                const unsigned long long w0 = wall_clock64();
                unsigned long long v[GANG_PARTS_MAX / 64], u[GANG_PARTS_MAX / 64];
                for (uint32_t spins = 0;;) {
                    bool all = true;
#pragma unroll
                    for (int q = 0; q < (int)GANG_PARTS_MAX / 64; ++q) {
                        const uint32_t b = tid + 64 * q;
                        v[q] = ((unsigned long long)want << 40) | 0xFFFFFFFFFFull;
                        u[q] = 0;
                        if (b < G) {
                            const unsigned long long *ln = kw + ((size_t)par * G + b) * KEY_STRIDE;
                            v[q] = __hip_atomic_load(ln, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            u[q] = __hip_atomic_load(ln + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                    }
#pragma unroll
                    for (int q = 0; q < (int)GANG_PARTS_MAX / 64; ++q)
                        all = all && (v[q] >> 40) == want &&
                              ((v[q] & 0xFFFFFFFFFFull) == 0xFFFFFFFFFFull || (u[q] >> 32) == seq);
                    if (__all(all)) break;
                    if ((++spins & 63u) == 0u && wall_clock64() - w0 > GANG_TICKS) {
                        sh.err = 1u;
                        break;
                    }
                }
                // least (iteration, order bits), the lowest part among equal
                // ones: as (iteration, high half) and (low half, part)
                unsigned long long bh = ~0ull, bl = ~0ull;
#pragma unroll
                for (int q = 0; q < (int)GANG_PARTS_MAX / 64; ++q) {
                    const unsigned long long h = v[q] & 0xFFFFFFFFFFull, l = (u[q] << 32 >> 24) | (tid + 64 * q);
                    if (h != 0xFFFFFFFFFFull && (h < bh || (h == bh && l < bl))) {
                        bh = h;
                        bl = l;
                    }
                }
                const unsigned long long have = __ballot(bh != ~0ull);
                if (have) {
                    if ((have & (have - 1)) == 0) {
                        const int l = __builtin_ctzll(have);
                        bh = (unsigned long long)__shfl((long long)bh, l, 64);
                        bl = (unsigned long long)__shfl((long long)bl, l, 64);
                    } else {
#pragma unroll
                        for (int off = 32; off >= 1; off >>= 1) {
                            const unsigned long long h = (unsigned long long)__shfl_xor((long long)bh, off, 64);
                            const unsigned long long l = (unsigned long long)__shfl_xor((long long)bl, off, 64);
                            if (h < bh || (h == bh && l < bl)) {
                                bh = h;
                                bl = l;
                            }
                        }
                    }
                    const uint32_t owner = (uint32_t)(bl & 0xFF);
                    const unsigned long long *src = pw + ((size_t)par * G + owner) * pstride;
                    const unsigned long long *srci = kw + ((size_t)par * G + owner) * KEY_STRIDE + 2;
                    for (uint32_t q0 = 0; q0 < pstride; q0 += 128) {
                        unsigned long long pv[2], pi;
                        for (uint32_t spins = 0;;) {
                            pi = __hip_atomic_load(srci, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                            for (int e = 0; e < 2; ++e) {
                                const uint32_t q = q0 + 64 * e + tid;
                                pv[e] = q < pstride
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
                            if (q < pstride) reinterpret_cast<uint32_t *>(s_gn)[q] = (uint32_t)pv[e];
                        }
                        if (tid == 0) sh.win_idx = (uint32_t)pi;
                    }
                }
                if (tid == 0) {
                    sh.win_hi = bh;
                    sh.win_lo = (uint32_t)(bl >> 8);
                }
            }
            __syncthreads();
            if (sh.err) break; // uniform; the state is lost and the caller told
            changed = sh.win_hi != ~0ull;
            nc = (uint32_t)(sh.win_hi >> 32);
            kk = (sh.win_hi << 32) | sh.win_lo;
            loc = sh.win_idx;
        } else {
            if (changed) { // uniform
                if (valid && j == loc) {
#pragma unroll
                    for (int q = 0; q < C; ++q)
                        if (d0 + q < D) s_gn[d0 + q] = S.x[q];
                }
                __syncthreads();
            }
        }
        if (!changed) nc = (uint32_t)n; // iterations committed
        if constexpr (SPEC) {
            // ran past the change: repeat its nc iterations from the block's
            // start, with the gbest of then
            if (changed && ran != nc) {
                S = B;
                for (uint32_t s = 1; s <= nc; ++s) {
                    if constexpr (MULTI) row ^= 1; // the rows are written again
                    iterate(tb + s, row, cand, ord);
                }
            }
        }
        if (changed) {
            gord = kk;
            gidx = loc;
            giter = t0 + done + nc;
            double *s_old = s_g;
            s_g = s_gn;
            s_gn = s_old;
        }
        done += nc;
        K = SPEC ? next_block(changed, (int)nc, ga.block_ratio, mean, since) : 1;
        stop = tol > 0.0 && fabs(ord64_value(gord) - fstar) < tol;
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
    if (tid == 0 && sh.err) atomicOr(&c->err, 1u);
    if (part != 0) return;
    for (int d = (int)tid; d < D; d += (int)T) a.gpos[d] = s_g[d];
    if (tid == 0) {
        c->gord = gord;
        c->gidx = gidx;
        c->giter = giter;
        c->t = t0 + done;
        c->stop = stop ? 1u : 0u;
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
struct Gang64Kernel {
    const void *fn;
    int C, max_lanes, pl;
    bool multi, uni;
};

template <int FIT, int C, bool MULTI, bool UNI, bool SPEC, int MAXT, int PL = 0>
static Gang64Kernel gang64_entry()
{
    return Gang64Kernel{reinterpret_cast<const void *>(k_gang64_resident<FIT, C, MULTI, UNI, SPEC, MAXT, PL>), C, MAXT,
                        PL, MULTI, UNI};
}

template <int FIT>
static const Gang64Kernel *gang64_table(int *n)
{
    // Double cos and exp leave 1024 lanes too few registers for C = 8; C = 4 spills
    // there too (42 to 80 registers, without them 6 to 9), C = 8 61 without them, and
    // C = 32 128 to 148 at 512 lanes (2 to 4 without).
    constexpr int MOST8 = FIT == F_RASTRIGIN || FIT == F_ACKLEY ? 512 : 1024;
    static const Gang64Kernel t[] = {
        gang64_entry<FIT, 1, false, true, true, 1024>(),
        gang64_entry<FIT, 2, false, true, true, 1024>(),
        gang64_entry<FIT, 4, false, true, true, 512>(),
        gang64_entry<FIT, 4, false, true, false, 1024>(),
        gang64_entry<FIT, 8, false, true, true, 512>(),
        gang64_entry<FIT, 16, false, true, false, 512>(),
        gang64_entry<FIT, 32, false, true, false, 512, 16>(),
        gang64_entry<FIT, 2, true, true, true, 1024>(),
        gang64_entry<FIT, 4, true, true, false, 1024>(),
        gang64_entry<FIT, 8, true, true, false, MOST8>(),
        gang64_entry<FIT, 16, true, true, false, 512>(),
        gang64_entry<FIT, 32, true, true, false, 512, 8>(),
        gang64_entry<FIT, 2, true, false, true, 1024>(),
        gang64_entry<FIT, 4, true, false, false, 1024>(),
        gang64_entry<FIT, 8, true, false, false, 512>(),
    };
    *n = (int)(sizeof t / sizeof t[0]);
    return t;
}

static const Gang64Kernel *gang64_kernels(int fitness, int *n)
{
    switch (fitness) {
    case F_SPHERE: return gang64_table<F_SPHERE>(n);
    case F_RASTRIGIN: return gang64_table<F_RASTRIGIN>(n);
    case F_ROSENBROCK: return gang64_table<F_ROSENBROCK>(n);
    case F_ACKLEY: return gang64_table<F_ACKLEY>(n);
    default: return gang64_table<F_CUBIC>(n);
    }
}

bool gang64_accepts(int fitness, const Swarm64Args &a)
{
    if (fitness < F_SPHERE || fitness > F_CUBIC) return false;
    auto minus_zero = [](double b) { return b == 0.0 && std::signbit(b); };
    return !minus_zero(a.lo) && !minus_zero(a.hi);
}

size_t gang64_words(uint64_t N, int D)
{
    if (D > GANG64_MAX_D_ALL) return 0;
    const uint64_t parts = std::min<uint64_t>(GANG_PARTS_MAX, (N + 15) / 16);
    return parts < 2 ? 0 : (size_t)(2 * parts * KEY_STRIDE + 2 * parts * 2 * (uint64_t)D);
}

static bool gang64_layout(int fitness, const Swarm64Args &a, int cus, int lds_max, int C, uint32_t P, Gang64Shape *out)
{
    int nk = 0;
    const Gang64Kernel *tab = gang64_kernels(fitness, &nk);
    const uint32_t L = ((uint32_t)a.D + C - 1) / C;
    const uint64_t lanes = ((uint64_t)P * L + 63) / 64 * 64, G = ((uint64_t)a.N + P - 1) / P;
    if (G > GANG_PARTS_MAX || G > (uint64_t)cus || (G > 1 && a.D > GANG64_MAX_D_ALL)) return false;
    if (P < 16) return false;
    for (int q = 0; q < nk; ++q) {
        const Gang64Kernel &kn = tab[q];
        if (kn.C != C || kn.multi != (L > 1) || lanes > (uint64_t)kn.max_lanes) continue;
        if (kn.uni != (P % 64 == 0)) continue;
        const int W = fitness == F_ACKLEY ? 2 : 1;
        size_t f = 3 * (size_t)L * C + lanes * (kn.pl ? kn.pl + 1 : 0);
        if (kn.multi) f += (size_t)W * (C + 1) * (L - 1) * P + (P + 1) / 2;
        if (kn.multi && fitness == F_ROSENBROCK) f += (size_t)(L - 1) * P;
        const size_t lds = sizeof(double) * f;
        if (lds + sizeof(Gang64Shared) + 1024 > (size_t)lds_max) continue;
        *out = Gang64Shape{kn.fn, C, P, L, (uint32_t)G, (uint32_t)lanes, lds};
        return true;
    }
    return false;
}

// The shape, as gang_shape chooses it in binary32 (pso_gang.hip), with smaller
// chunks, since an iteration of a dimension takes more.  Measured (us per
// iteration of the shape taken / the best of the others / the paths below the
// gang): one part: Rastrigin N = 100, D = 7 2.9 / 3.5 / 4.6, Cubic 128, 16
// 2.3 / 2.7 / 5.2, 32, 64 3.3 / 3.6 / 8.4; D = 1: Cubic N = 16384 0.84 / 0.87 /
// 7.4 (3.4 as a gang with its state in LDS that met every iteration); D <= 16:
// Rastrigin 4000, 7 5.1 / 5.2 / 13.1, Rosenbrock 8192, 12 4.2 / 4.6 / 12.0; D
// <= 64: Rastrigin 4000, 30 6.5 / 6.8 / 24.2, Cubic 16384, 64 8.4 / 9.4 / 24.1;
// beyond: Cubic 1000, 120 6.4 / 6.8 / 13.4, Rosenbrock 8192, 120 10.4 / 12.0 /
// 24.5; larger chunks: Cubic 16384, 120 C = 8 12.9 / 14.1 / 32.5; Rosenbrock
// 32768, 120 C = 32 16.9 / - / 46.4, Rastrigin 65536, 30 C = 16 15.6 / 24.7 (C =
// 8, which spills) / 40.8.
bool gang64_shape(int fitness, const Swarm64Args &a, int64_t t0, int64_t T, Gang64Shape *out)
{
    int cus = 0, lds_max = 0;
    if (!gang_device(&cus, &lds_max)) return false;
    auto layout = [&](int c, uint32_t P, Gang64Shape *s) { return gang64_layout(fitness, a, cus, lds_max, c, P, s); };
    if (const char *env = getenv("PSO64_GANG_SHAPE")) { // "C,P": forced (tests, measurements)
        int c = 0, p = 0;
        return sscanf(env, "%d,%d", &c, &p) == 2 && c >= 1 && p >= 16 && p <= 1024 &&
               layout(c, (uint32_t)p, out);
    }
    const int D = a.D;
    const uint32_t N = a.N;
    // double cos and exp: lanes of few dimensions, in several parts sooner
    const bool heavy = fitness == F_RASTRIGIN || fitness == F_ACKLEY;
    // Sphere and Rosenbrock improve their gbest for long (settles_late) and stay in
    // one part (us of 1000 iterations, one part / more / the paths below: Sphere
    // D = 2, N = 641 1535 / 1797 / 1694, N = 1024 1789 / 1774 / 1932; Rosenbrock D = 3,
    // N = 800 2490 / 2953 / 2648); Rastrigin and Ackley leave it at once, a brief run
    // of Cubic stays (of 100 iterations, Ackley N = 900, D = 1 339 / 269 / 329).
    const bool late = settles_late(fitness), brief = t0 + T < 200;
    const uint32_t most2 = heavy ? 640 : brief ? 1024 : late && D == 2 ? 768 : 640;
    const uint32_t most4 = late ? 1024 : brief ? 960 : 768;
    if (one_part(N, D, most2, most4, 0, [&](int c, uint32_t P) {
            return !(heavy && D > 2 && c > 2) && layout(c, P, out);
        }))
        return true;
    if (heavy && D > 12 && D <= 64) { // one_part starts with larger chunks there
        const uint32_t packed = std::max(16u, (N + 3) / 4 * 4);
        if (packed * ((uint32_t)(D + 1) / 2) <= 1024 && layout(2, packed, out)) return true;
    }
    int c = D == 1 ? 1 : 2;
    uint32_t pmin = 256, parts = 128;
    if (D <= 2) parts = 256;
    else if (D <= 4) c = N < 6000 ? 2 : 4, pmin = N < 6000 ? 32 : 256;
    else if (D <= 16) c = N < 6000 ? 2 : 4, pmin = N < 6000 ? 16 : 64;
    else if (heavy && D <= 64 && N < 6000) c = 2, pmin = 16;
    else if (D <= 64 || (N < 2000 && !heavy)) c = 4, pmin = N < 2000 ? 16 : 64;
    else c = 8, pmin = 16, parts = 256;
    for (; c <= 32; c *= 2) {
        const uint32_t L = ((uint32_t)D + c - 1) / c;
        uint32_t P = c >= 16 ? std::max(pmin, 64u) : pmin;
        if (L == 1) P = std::max(P, 64u);
        Gang64Shape s;
        bool ok = layout(c, P, &s);
        // more particles of a part while there are too many parts
        while (P < 1024 && (a.N + P - 1) / P > parts) {
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

hipError_t launch_gang64(int fitness, const Swarm64Args &a, const Gang64Shape &s, uint32_t T, hipStream_t stream)
{
    int cus = 0, lds_max = 0;
    if (!gang_device(&cus, &lds_max)) return hipErrorInvalidDevice;
    // the most any swarm may ask for, so concurrent callers never lower it
    hipError_t e = hipFuncSetAttribute(s.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       lds_max - (int)sizeof(Gang64Shared) - 1024);
    if (e != hipSuccess) return e;
    Swarm64Args args = a;
    Gang64Args ga{};
    ga.T = T;
    ga.P = s.P;
    ga.L = s.L;
    ga.c1s = std::ldexp(a.c1, -24);
    ga.c2s = std::ldexp(a.c2, -24);
    ga.words = a.gang_words;
    // double cos and exp: several times an iteration of the others
    ga.block_ratio = block_ratio(s.C, s.L, s.lanes, s.G, fitness == F_RASTRIGIN || fitness == F_ACKLEY ? 4.5f : 1.5f);
    void *params[] = {&args, &ga};
    return hipLaunchKernel(s.fn, dim3(s.G), dim3(s.lanes), params, s.lds, stream);
}

} // namespace pso
