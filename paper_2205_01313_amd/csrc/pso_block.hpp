// pso_block.hpp -- per-swarm workgroup kernels: a small swarm's whole run,
// and many swarms in one persistent launch (large swarms split into parts).
#pragma once

#include "pso_kernels.hpp"

namespace pso {

constexpr uint32_t MAX_PARTS = 64;         // workgroups one streamed batched swarm may span
constexpr uint32_t MAX_STAGED_PARTS = 512; // workgroups one LDS-staged batched swarm may span

// Value of a shape's stage_kib for parts that hold their particles in vector
// registers (pso_resident.hip): 256 lanes, L of them to a particle, each with
// cs dimensions; P particles of a part, a multiple of 64, so that the chunk is
// the same over a wavefront.  Small swarms take more lanes of fewer dimensions,
// and 33 to 48 dimensions four lanes rather than three, so that their parts
// fill their workgroups.
constexpr int STAGE_REGISTERS = 1 << 20;
constexpr int RESIDENT_LANES = 256, RESIDENT_C = 16, RESIDENT_MAX_D = 64;
constexpr int RESIDENT_PER_CU = 4;    // workgroups that share a compute unit
constexpr uint32_t RESIDENT_LINE = 8; // 64-bit words between the key words of two parts
struct ResidentSplit {
    uint32_t L, cs, P, parts;
};
__host__ __device__ inline ResidentSplit resident_split(uint64_t N, int D)
{
    uint32_t L = ((uint32_t)D + RESIDENT_C - 1) / RESIDENT_C;
    const uint32_t wide = N <= 64 ? 4u : N <= 128 ? 2u : 1u, most = (uint32_t)D / 4;
    if (L < wide && most > L) L = wide < most ? wide : most;
    if (L == 3) L = 4;
    uint32_t cs = ((uint32_t)D + L - 1) / L;
    cs += cs & 1u;
    L = ((uint32_t)D + cs - 1) / cs;
    const uint32_t P = L == 1 ? 256u : L == 2 ? 128u : 64u;
    return ResidentSplit{L, cs, P, (uint32_t)((N + P - 1) / P)};
}
// Whether holding a swarm of `parts` parts in registers beats staging it in
// LDS, in a launch of `total` parts in all on `grid` workgroups (registers
// against LDS in ms, 200 iterations of Rastrigin where nothing else is said):
//  - Parts that have a compute unit to themselves: a swarm of one or two parts
//    is faster on the 1024 lanes of the LDS-staged kernel (one swarm, D = 30,
//    N = 200: 1.17 against 1.00; N = 16: 0.66 / 0.48), as is one that is several
//    parts here, which meet, and one there (D <= 2, N = 1000: 0.42 / 0.35; 100
//    iterations, D = 3: N = 128 1.15 of LDS's time, 300 1.46, 640 1.24; D = 8: 300
//    1.43, 512 1.10; D = 16: 300 1.39), unless it is one part and D <= 2 (N = 200:
//    0.95 of it).  Larger swarms gain from being split further (100 iterations,
//    N = 1024: D = 3 0.93, 8 0.70; N = 640: D = 8 1.01, 16 0.91; N = 300, D = 20 0.98;
//    N = 200, D = 40 0.89).
//  - Parts that outnumber the workgroups at D <= 4: a register part holds 256
//    particles, an LDS part thousands, and meets as often (300 swarms of
//    N = 16000, D = 1: 18.0 / 9.4; D = 4: 20.0 / 18.3; D = 6: 0.88 of it).
//  - Else registers: 300 swarms of N = 1000, D = 30: 0.71 of LDS's time;
//    N = 200, D = 30: 0.91.
inline bool registers_pay(uint64_t N, int D, uint64_t parts, uint64_t total, int grid)
{
    if (total <= (uint64_t)(grid / RESIDENT_PER_CU)) {
        if (D <= 2) return N <= 256 || N > 1024;
        return D <= RESIDENT_C ? N > (D <= 8 ? 640 : 512) : N > 256 || parts > 2;
    }
    return !(D <= 4 && parts > 1 && total > (uint64_t)grid);
}

// Meeting point of the parts of one swarm (parts > 1): each part posts its
// workgroup-minimum key and, if it has one, that particle's position into the
// slots of the step's parity, as words tagged with the step (cand_key,
// cand_pos); err records a part that waited past the time bound.  The arrival
// count serves no meeting and stays zero.
struct GangSync {
    unsigned long long arrive;
    unsigned int err;
    unsigned int pad;
};

// One swarm of a batch: its state view (pointers into the batch's memory,
// parameters, Philox key), its run limits and, when split into parts, the
// parts' meeting point: cand_key[2][parts][2] (a key's low and high halves;
// of parts held in registers [2][parts][RESIDENT_LINE]) and
// cand_pos[2][parts][D] (one coordinate's bits), 64-bit words whose high
// halves carry the step.
struct BatchItem {
    SwarmArgs a;
    int32_t fitness;
    uint32_t parts;
    long long max_iter;
    float tol, fstar;
    GangSync *gang;
    unsigned long long *cand_key;
    float *cand_pos;
};

// Tiles and schedule of a batched launch: lanes per workgroup, co-resident
// workgroups, particle-dimension updates per part and iteration when a large
// swarm is split into parts, and the state's home during a launch.
// stage_kib = 0 streams every part's state from device memory each
// iteration (lanes 64, 128 or 256; parts by part_work); stage_kib > 0 copies
// each part's state into stage_kib KiB of LDS for the whole launch and
// splits swarms into as many parts as that takes (lanes 256, 512 or 1024;
// part_work unused).  Every shape computes the same bits; only the time
// differs.
struct BatchShape {
    int lanes;
    int grid;
    long long part_work;
    int stage_kib;
};
constexpr BatchShape DEFAULT_BATCH_SHAPE = {256, 0, 1 << 17, 0}; // grid 0: the co-resident capacity
// A batch's shape before any autotuning when every swarm fits it (else the
// streamed default): one 1024-lane workgroup per compute unit with 158 KiB
// of staged state (less where the batch's widest D needs more LDS room).
constexpr BatchShape DEFAULT_STAGED_SHAPE = {1024, 0, 0, 158};

bool batch_lanes_supported(int lanes, bool staged = false);

// LDS bytes one staged particle quad takes: x, v, p and the fitness terms of
// each of D dimensions, its pbest fitness and pending marks.
size_t staged_quad_bytes(int D, int fitness);

// Parts of a swarm under an LDS-staged shape (each part's quads fit
// stage_kib KiB), or 0 if it would need more than MAX_STAGED_PARTS or
// grid_cap workgroups.
uint32_t staged_parts(uint64_t N, int D, int fitness, int stage_kib, int grid_cap);

// Parts for a batched swarm: about one part per shape.part_work
// particle-dimension updates of an iteration, at least one particle quad per
// lane of a part, at most MAX_PARTS and at most grid_cap (the workgroups of
// the launches it joins).
uint32_t parts_for(uint64_t N, int D, int grid_cap, const BatchShape &shape);

// Bytes of a swarm's gang region for `parts` parts (0 when parts == 1).
size_t gang_bytes(uint32_t parts, int D);
// Points the item's gang fields into a region of gang_bytes(parts, D).
void bind_gang(BatchItem *it, void *region, uint32_t parts);
// The same for parts held in registers: each part's key words on a line of
// their own.
inline size_t resident_gang_bytes(uint32_t parts, int D)
{
    const size_t words = sizeof(unsigned long long) * 2 * parts * (size_t)(RESIDENT_LINE + D);
    return parts <= 1 ? 0 : 256 + ((words + 255) & ~size_t(255));
}
inline void bind_resident_gang(BatchItem *it, void *region, uint32_t parts)
{
    it->parts = parts < 1 ? 1 : parts;
    it->gang = nullptr;
    it->cand_key = nullptr;
    it->cand_pos = nullptr;
    if (it->parts == 1) return;
    it->gang = static_cast<GangSync *>(region);
    it->cand_key = reinterpret_cast<unsigned long long *>(static_cast<char *>(region) + 256);
    it->cand_pos = reinterpret_cast<float *>(it->cand_key + 2 * (size_t)parts * RESIDENT_LINE);
}

// Loop state (and result) of one batched swarm, kept in device memory
// between launches; the gbest position is kept in a.gpos.
struct BatchResult {
    unsigned long long gkey; // gbest key (fitness, index)
    long long giter;         // iteration of the last gbest change
    long long iters;         // iterations run
    uint32_t started;        // Step 1 done
    uint32_t stop;           // stop rule met
    uint32_t ticks;          // device wall-clock ticks of the last launch's share (part 0)
    uint32_t pad;
};

// One unit of a batched launch: part `part` of item `item`; the item's state
// is also copied to position `out` of the launch's compact outputs.  iters > 0
// fixes the iterations of this launch for the swarm (every part of a swarm
// carries the same value); 0 takes the `chunk` rule of launch_batch.
struct BatchEntry {
    uint32_t item, part, out, iters;
};

// Runs up to T more iterations of one swarm in one workgroup, continuing from
// and updating its control block (stop rule included): its state staged in
// LDS where it fits (or PSO_BLOCK_STAGED=0 in the environment), else read
// from device memory every iteration.
hipError_t launch_block_run(int fitness, const SwarmArgs &a, long long T, hipStream_t stream);
// Whether a pso_run of this swarm should take the one-workgroup run: its
// state fits one workgroup's LDS (always true under PSO_BLOCK_STAGED=0).
bool block_run_suits(int fitness, const SwarmArgs &a);
// Marks results[0..count) not started (and their gangs unused); clears the
// work counter.
hipError_t launch_batch_reset(const BatchItem *items, BatchResult *results, uint32_t count, unsigned int *next,
                              hipStream_t stream);

// One persistent launch of `grid` workgroups over `count` entries (every part
// of a listed swarm, consecutive): Step 1 for swarms not started, then the
// entry's iters, or clamp(chunk / (N*D), 1, iter_cap), more iterations of
// each -- `chunk` is a budget of particle-dimension updates per swarm and
// launch -- within its max_iter and stop rule.  `next` is a device work counter (cleared by the launch).  The
// grid must be fully co-resident (at most batch_capacity workgroups, less
// any other launch running concurrently) and every swarm's parts <= grid.
// Optionally writes each swarm's state to out_state[out] and its gbest
// position to out_pos[out*maxD ..]; device errors set *err.
// stage_kib > 0 runs the LDS-staged kernel, STAGE_REGISTERS the one that holds
// parts in registers (every item's parts must come from staged_parts for the
// same stage_kib).
hipError_t launch_batch(const BatchItem *items, const BatchEntry *entries, BatchResult *results, uint32_t count,
                        unsigned int *next, int maxD, int grid, int lanes, long long chunk, long long iter_cap,
                        hipStream_t stream, BatchResult *out_state, float *out_pos, unsigned int *err,
                        int stage_kib = 0);
// launch_batch for STAGE_REGISTERS, the workgroups of it a compute unit holds,
// and its LDS.
hipError_t launch_batch_resident(const BatchItem *items, const BatchEntry *entries, BatchResult *results, uint32_t count,
                                 unsigned int *next, int grid, long long chunk, long long iter_cap, hipStream_t stream,
                                 BatchResult *out_state, float *out_pos, int pos_stride, unsigned int *err);
hipError_t resident_occupancy(int *per_cu);
size_t resident_lds();
// Workgroups of `lanes` lanes of the batched kernel (LDS-staged with
// stage_kib KiB if > 0) that are safely co-resident: three quarters of the
// occupancy bound streamed, all but 8 compute units' worth staged; 0 if the
// staged LDS does not fit a workgroup.
hipError_t batch_capacity(int maxD, int lanes, int *workgroups, int stage_kib = 0);
// LDS bytes a workgroup of the batched kernel takes dynamically.
size_t batch_dynamic_lds(int maxD, int stage_kib);

// Staged KiB per workgroup that leave room, in a compute unit's LDS shared
// by per_cu workgroups, for each workgroup's gbest position and shift of
// maxD floats: at most 158 (per_cu = 1) or 78 (per_cu = 2); 0 if none fit.
int staged_kib_fitting(int maxD, int per_cu);
// Workgroups a launch of this shape takes: grid > 0 as given (at most the
// co-resident capacity), 0 the capacity, -k the capacity / k; 0 if a staged
// shape's LDS does not fit a workgroup.
hipError_t shape_grid(int maxD, const BatchShape &sh, int *grid);
// Sets one device word to zero with a kernel (stream-ordered; no memset).
hipError_t launch_clear_u32(unsigned int *p, hipStream_t stream);

// The first upload of a newly admitted request to the request server's
// device tables: its item and loop state go to slot `slot`, its D shift
// floats (from a launch's float pool, at shift_at) to item.a.shift, and a
// swarm of several parts gets its gang counters cleared.  One record per
// request; launch_upload applies a launch's records in one kernel, so the
// uploads of a launch are two copies and one launch whatever their number.
struct UploadRec {
    BatchItem item;
    BatchResult state;
    uint32_t slot;
    uint32_t shift_at;
    uint32_t reset_gang;
    uint32_t pad;
};
hipError_t launch_upload(const UploadRec *recs, uint32_t n, const float *pool, BatchItem *items, BatchResult *state,
                         hipStream_t stream);

} // namespace pso
