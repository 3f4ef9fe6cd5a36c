// Row bands (ising_band_rows.hpp): the Metropolis kernels, and the shapes in
// which either dynamics is served.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_band_rows.hpp"

namespace ising {

namespace {

template <int CW, int MODE>
const void* kernel_d(uint32_t d) {
    if (d == 1u) return reinterpret_cast<const void*>(&k_band_rows<CW, MODE, 1, false>);
    if (d == 2u) return CW <= 6 ? reinterpret_cast<const void*>(&k_band_rows<CW <= 6 ? CW : 1, MODE, 2, false>) : nullptr;
    return CW <= 4 ? reinterpret_cast<const void*>(&k_band_rows<CW <= 4 ? CW : 1, MODE, 4, false>) : nullptr;
}
template <int MODE>
const void* kernel_cw(uint32_t cw, uint32_t d) {
    switch (cw) {
        case 1: return kernel_d<1, MODE>(d);
        case 2: return kernel_d<2, MODE>(d);
        case 3: return kernel_d<3, MODE>(d);
        case 4: return kernel_d<4, MODE>(d);
        case 5: return kernel_d<5, MODE>(d);
        case 6: return kernel_d<6, MODE>(d);
        case 7: return kernel_d<7, MODE>(d);
        case 8: return kernel_d<8, MODE>(d);
        default: return nullptr;
    }
}

}  // namespace

const void* row_band_kernel(const RowBandShape& s) {
    if (s.creutz) return creutz_row_kernel(s);
    return s.mode == kRowsFull ? kernel_cw<kRowsFull>(s.cw, s.depth)
           : s.mode == kRowsRagged ? kernel_cw<kRowsRagged>(s.cw, s.depth) : kernel_cw<kRowsShifted>(s.cw, s.depth);
}

// Row layout of side L: words a lane and how rows end.
static bool row_layout(uint32_t L, uint32_t* cw, uint32_t* mode) {
    const uint32_t H2 = L / 2u;
    if (L % 8u == 0u) {
        const uint32_t Hw = H2 / 4u;
        if (Hw % 64u == 0u) {
            *cw = Hw / 64u;
            *mode = kRowsFull;
        } else {
            *cw = Hw / 64u + 1u;  // the ghost word fits: Hw + 1 <= 64 cw
            *mode = kRowsRagged;
        }
    } else {
        // up to 3 bytes before the first site, one ghost byte after the last
        const uint32_t words = (3u + H2) / 4u + 1u;
        *cw = (words + 63u) / 64u;
        *mode = kRowsShifted;
    }
    return *cw >= 1u && *cw <= 8u;
}

bool row_band_shape(uint32_t L, uint32_t G, bool creutz, RowBandShape* out) {
    if (L < 4u || (L & 1u) || G < 2u || G > L) return false;
    RowBandShape s;
    s.creutz = creutz;
    if (!row_layout(L, &s.cw, &s.mode)) return false;
    const uint32_t hmax = (L + G - 1u) / G, hmin = L / G;
    for (s.depth = 4u; s.depth >= 1u; s.depth /= 2u) {
        if (s.depth > hmin || hmax + 2u * (s.depth - 1u) > kMaxRowWaves || !row_band_kernel(s)) continue;
        s.threads = 64u * (hmax + 2u * (s.depth - 1u));
        s.lds = row_band_lds_words(s.threads / 64u, s.cw) * 4u;
        *out = s;
        return true;
    }
    return false;
}

size_t row_band_pub_words(uint32_t L, uint32_t G, bool creutz) {
    RowBandShape s;
    if (!row_band_shape(L, G, creutz, &s)) return 0;
    return (size_t)2 * G * 2u * s.depth * (size_t)entries_per_row((int)s.cw, (int)s.depth, creutz) * 64u + G;
}

}  // namespace ising
