// Tagged words in global memory with which the workgroups of a band launch
// trade their edge rows (ising_bands.hip, ising_band_rows.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ising {
namespace {

// Polls of an edge word (each a read of its coherent copy and a short sleep)
// before a wait gives up: several seconds.
constexpr uint32_t kBandMaxPolls = 1u << 24;

__device__ __forceinline__ void put_word(uint64_t* p, uint32_t tag, uint32_t w) {
    __hip_atomic_store(p, ((uint64_t)tag << 32) | w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The words at p[0 .. N-1] once their tags are `tag` (the whole wave waits
// until every lane's words have it). All N are read in every poll: their
// latencies overlap. *err (host memory) is looked at only in long waits.
template <int N>
__device__ __forceinline__ void take_words(const uint64_t* const (&p)[N], uint32_t tag, uint32_t* err,
                                           uint32_t (&out)[N]) {
    uint32_t polls = 0;
    for (;;) {
        uint64_t v[N];
        uint32_t miss = 0;
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = __hip_atomic_load(p[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            out[k] = (uint32_t)v[k];
            miss |= (uint32_t)(v[k] >> 32) ^ tag;
        }
        if (__ballot(miss != 0u) == 0) break;
        if ((++polls & 255u) == 0u) {
            if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) break;
            if (polls >= kBandMaxPolls) {
                __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                break;
            }
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

__device__ __forceinline__ uint32_t take_word(const uint64_t* p, uint32_t tag, uint32_t* err) {
    const uint64_t* const ps[1] = {p};
    uint32_t v[1];
    take_words<1>(ps, tag, err, v);
    return v[0];
}

}  // namespace
}  // namespace ising
