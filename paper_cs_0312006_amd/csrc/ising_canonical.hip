// Layout conversion between colour planes and canonical row-major bytes:
// spins (planes 1 / 0, canonical +1 / -1) and plain bytes (demons).
//
// Site j of row i is byte j >> 1 of plane (i + j) & 1, so a canonical row is
// the bytes of plane i & 1 (even columns) and of the other plane (odd
// columns) in turn: two byte permutes a word pair. Bound by memory (each byte
// read and written once): with four words of each plane a thread, 16384^2
// takes 0.09 ms and 32768^2 0.46 ms (4.6 TB/s), against 0.54 and 2.03 ms with
// a thread a site (a 64-bit division and a byte load and store each). The
// site kernels stay for sides of partial words and for buffers that are not
// aligned for the wider accesses.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_device.hpp"
#include "ising_launch.hpp"

namespace ising {

namespace {

constexpr uint32_t kThreads = 256;

template <bool SPINS>
__device__ __forceinline__ uint32_t to_canon(uint32_t v) {
    return SPINS ? ~(v * 0xfeu) : v;  // bytes 1 -> 0x01, 0 -> 0xff
}
template <bool SPINS>
__device__ __forceinline__ uint32_t from_canon(uint32_t v) {
    return SPINS ? (~v >> 1) & 0x01010101u : v;  // 0x01 -> 1, 0xff -> 0
}

template <int W>
struct Words {
    uint32_t v[W];
};

template <int W, bool SPINS>
__global__ void __launch_bounds__(kThreads) k_words_to_canonical(Planes pl, uint32_t* __restrict__ out) {
    using V = __attribute__((ext_vector_type(W))) uint32_t;
    using V2 = __attribute__((ext_vector_type(2))) uint32_t;
    const uint32_t per_row = pl.Hw / W, total = pl.L * per_row, stride = gridDim.x * kThreads;
    for (uint32_t g = blockIdx.x * kThreads + threadIdx.x; g < total; g += stride) {
        const uint32_t odd = (g / per_row) & 1u;
        Words<W> a, b;  // even and odd columns
        if constexpr (W == 1) {
            a.v[0] = reinterpret_cast<const uint32_t*>(pl.p[odd])[g];
            b.v[0] = reinterpret_cast<const uint32_t*>(pl.p[odd ^ 1u])[g];
        } else {
            const V x = reinterpret_cast<const V*>(pl.p[odd])[g], y = reinterpret_cast<const V*>(pl.p[odd ^ 1u])[g];
#pragma unroll
            for (int w = 0; w < W; ++w) a.v[w] = x[w], b.v[w] = y[w];
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t x = to_canon<SPINS>(a.v[w]), y = to_canon<SPINS>(b.v[w]);
            const V2 o = {__builtin_amdgcn_perm(y, x, 0x05010400u), __builtin_amdgcn_perm(y, x, 0x07030602u)};
            reinterpret_cast<V2*>(out)[(size_t)g * W + w] = o;
        }
    }
}

template <int W, bool SPINS>
__global__ void __launch_bounds__(kThreads) k_words_from_canonical(Planes pl, const uint32_t* __restrict__ in) {
    using V = __attribute__((ext_vector_type(W))) uint32_t;
    using V2 = __attribute__((ext_vector_type(2))) uint32_t;
    const uint32_t per_row = pl.Hw / W, total = pl.L * per_row, stride = gridDim.x * kThreads;
    for (uint32_t g = blockIdx.x * kThreads + threadIdx.x; g < total; g += stride) {
        const uint32_t odd = (g / per_row) & 1u;
        Words<W> a, b;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const V2 v = reinterpret_cast<const V2*>(in)[(size_t)g * W + w];
            a.v[w] = from_canon<SPINS>(__builtin_amdgcn_perm(v.y, v.x, 0x06040200u));
            b.v[w] = from_canon<SPINS>(__builtin_amdgcn_perm(v.y, v.x, 0x07050301u));
        }
        if constexpr (W == 1) {
            reinterpret_cast<uint32_t*>(pl.p[odd])[g] = a.v[0];
            reinterpret_cast<uint32_t*>(pl.p[odd ^ 1u])[g] = b.v[0];
        } else {
            V x, y;
#pragma unroll
            for (int w = 0; w < W; ++w) x[w] = a.v[w], y[w] = b.v[w];
            reinterpret_cast<V*>(pl.p[odd])[g] = x;
            reinterpret_cast<V*>(pl.p[odd ^ 1u])[g] = y;
        }
    }
}

// Any even L, any alignment: a workgroup a row at a time, a thread a site.
template <bool SPINS>
__global__ void __launch_bounds__(kThreads) k_sites_to_canonical(Planes pl, uint8_t* __restrict__ out) {
    for (uint32_t i = blockIdx.x; i < pl.L; i += gridDim.x)
        for (uint32_t j = threadIdx.x; j < pl.L; j += kThreads) {
            const uint8_t v = pl.p[(i + j) & 1u][(size_t)i * pl.H + (j >> 1)];
            out[(size_t)i * pl.L + j] = SPINS ? (v ? 0x01u : 0xffu) : v;
        }
}

template <bool SPINS>
__global__ void __launch_bounds__(kThreads) k_sites_from_canonical(Planes pl, const uint8_t* __restrict__ in) {
    for (uint32_t i = blockIdx.x; i < pl.L; i += gridDim.x)
        for (uint32_t j = threadIdx.x; j < pl.L; j += kThreads) {
            const uint8_t v = in[(size_t)i * pl.L + j];
            pl.p[(i + j) & 1u][(size_t)i * pl.H + (j >> 1)] = SPINS ? (v == 0x01u ? 1u : 0u) : v;
        }
}

uint32_t blocks_for(uint64_t n) {
    const uint64_t b = (n + kThreads - 1) / kThreads;
    return (uint32_t)(b > 8192 ? 8192 : (b ? b : 1));
}

// Words a thread takes: four where rows are whole groups of four and both
// sides are aligned to them, one where words are aligned, else none.
int words_of(const Planes& pl, const void* canon) {
    if (pl.L % 8u != 0u) return 0;
    const uintptr_t p = reinterpret_cast<uintptr_t>(pl.p[0]) | reinterpret_cast<uintptr_t>(pl.p[1]);
    const uintptr_t c = reinterpret_cast<uintptr_t>(canon);
    if (pl.Hw % 4u == 0u && p % 16u == 0u && c % 8u == 0u) return 4;
    return p % 4u == 0u && c % 8u == 0u ? 1 : 0;
}

template <bool SPINS>
hipError_t to_canonical(const Planes& pl, void* out, hipStream_t s) {
    const uint64_t words = (uint64_t)pl.L * pl.Hw;
    switch (words_of(pl, out)) {
        case 4: k_words_to_canonical<4, SPINS><<<blocks_for(words / 4u), kThreads, 0, s>>>(pl, static_cast<uint32_t*>(out)); break;
        case 1: k_words_to_canonical<1, SPINS><<<blocks_for(words), kThreads, 0, s>>>(pl, static_cast<uint32_t*>(out)); break;
        default: k_sites_to_canonical<SPINS><<<pl.L > 8192u ? 8192u : pl.L, kThreads, 0, s>>>(pl, static_cast<uint8_t*>(out));
    }
    return hipGetLastError();
}

template <bool SPINS>
hipError_t from_canonical(const Planes& pl, const void* in, hipStream_t s) {
    const uint64_t words = (uint64_t)pl.L * pl.Hw;
    switch (words_of(pl, in)) {
        case 4: k_words_from_canonical<4, SPINS><<<blocks_for(words / 4u), kThreads, 0, s>>>(pl, static_cast<const uint32_t*>(in)); break;
        case 1: k_words_from_canonical<1, SPINS><<<blocks_for(words), kThreads, 0, s>>>(pl, static_cast<const uint32_t*>(in)); break;
        default: k_sites_from_canonical<SPINS><<<pl.L > 8192u ? 8192u : pl.L, kThreads, 0, s>>>(pl, static_cast<const uint8_t*>(in));
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_to_canonical(const Planes& pl, int8_t* out, hipStream_t s) { return to_canonical<true>(pl, out, s); }
hipError_t launch_from_canonical(const Planes& pl, const int8_t* in, hipStream_t s) { return from_canonical<true>(pl, in, s); }
hipError_t launch_bytes_to_canonical(const Planes& pl, uint8_t* out, hipStream_t s) { return to_canonical<false>(pl, out, s); }
hipError_t launch_bytes_from_canonical(const Planes& pl, const uint8_t* in, hipStream_t s) {
    return from_canonical<false>(pl, in, s);
}

}  // namespace ising
