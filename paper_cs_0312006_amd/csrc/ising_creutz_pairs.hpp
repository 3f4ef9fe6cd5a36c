// Two Creutz sweeps a launch (ising_creutz_pairs.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ising {

// Planes of the first (0) and second (1) colour of a sweep: a forward
// sweep's planes in order, a reversed sweep's exchanged.
struct CreutzPairArgs {
    const uint32_t* s0;  // spins before
    const uint32_t* s1;
    const uint32_t* m0;  // demons before
    const uint32_t* m1;
    uint32_t* d0;        // spins after
    uint32_t* d1;
    uint32_t* e0;        // demons after
    uint32_t* e1;
    uint32_t L, Hw, rows;
    int64_t* part;       // [2 sweeps][bands] (B, M)
};

struct CreutzPairShape {
    uint32_t cw, threads, rows, bands, lds;
    bool ragged;
};

// The launch for side L (L % 8 == 0, rows of at most 16 waves of four words a
// lane: L <= 32768) on a GPU of `cus` compute units; false if not served.
bool creutz_pairs_shape(uint32_t L, uint32_t cus, CreutzPairShape* out);
hipError_t launch_creutz_pair(const CreutzPairArgs& a, const CreutzPairShape& s, bool reverse, hipStream_t stream);

}  // namespace ising
