// Launchers of the percolation engine (perc_kernels.hip), shared with its
// runtime (perc_runtime.cpp).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace perc {

constexpr uint32_t kTile = 64;               // tile side (sites)
constexpr uint32_t kThreads = 256;           // per workgroup of the draw, seed and finish passes
constexpr uint32_t kRelaxThreads = 64;       // relaxation: one wave per tile
constexpr uint32_t kLevels = 32;             // arrival passes per relaxation launch (half a tile)
constexpr uint32_t kSubs = 64;               // parts of a work list, each with its own counter

// Summary of one medium's run.
struct Result {
    unsigned long long pores;
    unsigned long long invaded;
    uint32_t max_arrival;
    uint32_t edges;  // bit 0 row 0, bit 1 row L-1, bit 2 column 0, bit 3 column L-1
    unsigned long long visits;      // tile visits over all relaxation launches
    unsigned long long iterations;  // breadth-first levels summed over visits
};

struct TileStat {
    uint32_t visits, iterations, max_arrival, pad;
};

// One medium of a run (a run relaxes one or several media together). Bit
// maps are stored tile by tile: 64 rows of 64 bits (bit c: column c).
struct Medium {
    uint8_t* pore;        // row-major, 1 = pore
    uint32_t* arr;        // arrival passes, row-major (all ones: solid or not invaded)
    uint64_t* pmap;       // pores
    uint64_t* reach[2];   // invaded sites before launch k in reach[k % 2]
    uint32_t* queued[2];  // per tile: is it in work list 0 / 1
    TileStat* stat;       // per tile
    uint64_t pthr;        // a site is a pore iff its draw is below it
    uint32_t L, n_tx, n_ty;
    uint32_t k0, k1;      // Philox key
    uint32_t source, i0, j0;
};

// Work lists of (medium, tile) entries to relax in a launch. Launch k reads
// list[k % 2] with lengths len[k % 3], appends to list[(k + 1) % 2] /
// len[(k + 1) % 3] and clears len[(k + 2) % 3]; a medium's queued[p][tile]
// says whether the tile is in list p, so no tile is listed twice. A list has
// kSubs parts of `cap` entries: tile (ty, tx) of medium m goes to part
// (tx + 13 ty + m) % kSubs, so that a front's tiles, and those of small media of
// a batch, spread over the parts, their counters and the workgroups that read
// them (60 media of one tile each in part 0: 2.1 ms a run, spread 0.15).
struct WorkLists {
    uint2* list[2];
    uint32_t* len;  // 3 x kSubs counters
    uint32_t cap;
};
__host__ __device__ inline uint32_t list_part(uint32_t m, uint32_t tx, uint32_t ty) {
    return (tx + 13u * ty + m) % kSubs;
}
// Most entries of a side-L medium that go to one part.
__host__ __device__ inline uint64_t part_entries(uint32_t L) {
    const uint64_t n = (L + kTile - 1u) / kTile;
    return n * ((n + kSubs - 1u) / kSubs);
}

// Draw `count` media (max_L the largest side), clear their maps, flags and
// statistics, the list counters and the results.
hipError_t launch_draw(const Medium* media, uint32_t count, uint32_t max_L, const WorkLists& w, Result* res,
                       hipStream_t s);
// append every medium's source tiles to list 0
hipError_t launch_seed(const Medium* media, uint32_t count, const WorkLists& w, hipStream_t s);
// Relaxation launch k over the listed tiles; one: the host's descriptor when
// the run has a single medium (else nullptr).
hipError_t launch_relax(const Medium* one, const Medium* media, const WorkLists& w, uint64_t k, uint32_t grid,
                        hipStream_t s);
hipError_t launch_finish(const Medium* media, uint32_t count, uint32_t max_L, Result* res, hipStream_t s);

}  // namespace perc
