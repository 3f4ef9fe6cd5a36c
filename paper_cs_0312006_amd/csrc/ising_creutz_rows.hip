// Row bands (ising_band_rows.hpp): the Creutz kernels. Edges are traded every
// four half-sweeps where a band is at least four rows high and its rows take
// at most four words a lane, else every half-sweep.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_band_rows.hpp"

namespace ising {

namespace {

template <int MODE>
const void* kernel_cw(uint32_t cw, uint32_t d) {
    if (d == 4u) switch (cw) {
        case 1: return reinterpret_cast<const void*>(&k_band_rows<1, MODE, 4, true>);
        case 2: return reinterpret_cast<const void*>(&k_band_rows<2, MODE, 4, true>);
        case 3: return reinterpret_cast<const void*>(&k_band_rows<3, MODE, 4, true>);
        case 4: return reinterpret_cast<const void*>(&k_band_rows<4, MODE, 4, true>);
        default: return nullptr;
    }
    if (d == 1u) switch (cw) {
        case 1: return reinterpret_cast<const void*>(&k_band_rows<1, MODE, 1, true>);
        case 2: return reinterpret_cast<const void*>(&k_band_rows<2, MODE, 1, true>);
        case 3: return reinterpret_cast<const void*>(&k_band_rows<3, MODE, 1, true>);
        case 4: return reinterpret_cast<const void*>(&k_band_rows<4, MODE, 1, true>);
        case 5: return reinterpret_cast<const void*>(&k_band_rows<5, MODE, 1, true>);
        case 6: return reinterpret_cast<const void*>(&k_band_rows<6, MODE, 1, true>);
        case 7: return reinterpret_cast<const void*>(&k_band_rows<7, MODE, 1, true>);
        case 8: return reinterpret_cast<const void*>(&k_band_rows<8, MODE, 1, true>);
        default: return nullptr;
    }
    return nullptr;
}

}  // namespace

const void* creutz_row_kernel(const RowBandShape& s) {
    return s.mode == kRowsFull ? kernel_cw<kRowsFull>(s.cw, s.depth)
           : s.mode == kRowsRagged ? kernel_cw<kRowsRagged>(s.cw, s.depth) : kernel_cw<kRowsShifted>(s.cw, s.depth);
}

}  // namespace ising
