// Draws of sites a thread keeps for many sweeps (the row bands and the
// smallest resident lattices), and a wave sum without LDS.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_device.hpp"

namespace ising {
namespace {

// The parts of the Philox4x32-10 calls of quad q that do not depend on the
// sweep. With key (k0, k1), counter (q, t, c, 0) and W the key increments:
//   round 1: x = (t ^ k0, c M1, hi(M0 q) ^ k1, lo(M0 q))      (c < 2: hi(M1 c) = 0)
//   round 2: x = (hi(M1 x2) ^ c M1 ^ k0 + W0, lo(M1 x2), hi(M0 (t ^ k0)) ^ lo(M0 q) ^ k1 + W1, lo(M0 (t ^ k0)))
//   round 3: x = (hi(M1 x2) ^ x1 ^ k0 + 2 W0, lo(M1 x2), hi(M0 x0) ^ x3 ^ k1 + 2 W1, lo(M0 x0))
// so lo(M0 q) (a), the second round's x1 with round 3's key (b) and the
// third round's product M0 x0 (p, one for each colour) are fixed.
struct SiteDraws {
    uint32_t a, b;
};

__device__ __forceinline__ SiteDraws site_draws(uint32_t q, uint32_t k0, uint32_t k1, uint32_t& x0_c0) {
    const uint64_t p0 = mul_u64(q, kPhiloxM0);
    const uint64_t p1 = mul_u64((uint32_t)(p0 >> 32) ^ k1, kPhiloxM1);
    x0_c0 = (uint32_t)(p1 >> 32) ^ (k0 + kPhiloxW0);  // colour 0; colour 1: ^ M1
    return {(uint32_t)p0, (uint32_t)p1 ^ (k0 + 2u * kPhiloxW0)};
}

// The wave-uniform parts of a half-sweep's calls.
struct SweepDraws {
    uint32_t u, v;
};
__device__ __forceinline__ SweepDraws sweep_draws(uint32_t t, uint32_t k0, uint32_t k1) {
    const uint64_t p = (uint64_t)kPhiloxM0 * (t ^ k0);
    return {(uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) ^ (k1 + kPhiloxW1))),
            (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)p ^ (k1 + 2u * kPhiloxW1)))};
}

// Rounds FROM .. TO - 1 (of 0 .. 9) on the words x.
template <int FROM, int TO>
__device__ __forceinline__ uint4 philox_rounds(uint4 x, uint32_t k0, uint32_t k1) {
    k0 += (uint32_t)FROM * kPhiloxW0;
    k1 += (uint32_t)FROM * kPhiloxW1;
#pragma unroll
    for (int r = FROM; r < TO; ++r) {
        const uint64_t q0 = (uint64_t)kPhiloxM0 * x.x, q1 = (uint64_t)kPhiloxM1 * x.z;
        const uint32_t rk0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)k0);
        const uint32_t rk1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)k1);
        x = make_uint4(xor3((uint32_t)(q1 >> 32), x.y, rk0), (uint32_t)q1, xor3((uint32_t)(q0 >> 32), x.w, rk1),
                       (uint32_t)q0);
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
    }
    return x;
}

// The words after the third round from the fixed parts: p is M0 times the
// second round's x0.
__device__ __forceinline__ uint4 philox_third(const SiteDraws& f, uint64_t p, const SweepDraws& s) {
    const uint64_t p1 = mul_u64(f.a ^ s.u, kPhiloxM1);
    return make_uint4((uint32_t)(p1 >> 32) ^ f.b, (uint32_t)p1, (uint32_t)(p >> 32) ^ s.v, (uint32_t)p);
}

// The four draws.
__device__ __forceinline__ uint4 philox_fixed(const SiteDraws& f, uint64_t p, const SweepDraws& s, uint32_t k0,
                                              uint32_t k1) {
    return philox_rounds<3, 10>(philox_third(f, p, s), k0, k1);
}

// Sum over the wave, valid in lane 63 (whole-wave DPP reduction: no LDS
// round trips on the path between two barriers).
__device__ __forceinline__ uint32_t wave_sum_lane63(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

}  // namespace
}  // namespace ising
