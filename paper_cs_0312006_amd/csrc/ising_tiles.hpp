// One sweep a launch over wave tiles of any row length (ising_tiles.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_device.hpp"
#include "ising_launch.hpp"

namespace ising {

struct TileShape {
    uint32_t cw, rows, n_tx, tiles;
};

// The tiles of side L (L % 8 == 0).
bool tiles_shape(uint32_t L, TileShape* out);
// As launch_fused: a.n_tx and a.n_tiles are the shape's, a.part holds a pair
// a tile.
hipError_t launch_tiles(const FusedArgs& a, const AcceptTable& at, const TileShape& shape, const PartialReduce& red,
                        hipStream_t s);

}  // namespace ising
