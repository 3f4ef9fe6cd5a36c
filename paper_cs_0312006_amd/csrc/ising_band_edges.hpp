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

// The word at p once its tag is `tag` (the whole wave waits until every
// lane's word has it). *err (host memory) is looked at only in long waits.
__device__ __forceinline__ uint32_t take_word(const uint64_t* p, uint32_t tag, uint32_t* err) {
    uint64_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t polls = 0;
    while (__ballot((uint32_t)(v >> 32) != tag)) {
        if ((++polls & 255u) == 0u) {
            if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) break;
            if (polls >= kBandMaxPolls) {
                __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                break;
            }
        }
        __builtin_amdgcn_s_sleep(1);
        v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return (uint32_t)v;
}

}  // namespace
}  // namespace ising
