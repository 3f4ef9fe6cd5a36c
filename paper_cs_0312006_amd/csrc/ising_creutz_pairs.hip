// Two Creutz sweeps a launch, for lattices too large to stay on chip: spins
// and demons cross HBM once per two sweeps (2 bytes a site update, where one
// sweep a launch moves 4 and two in-place passes 5).
//
// What bounds the one-sweep launch is memory (0.96 of a copy's rate at 0.31
// of the vector units); this one halves the traffic. A workgroup of up to 16
// waves owns a band of whole rows and walks down it, a lane holding CW words
// of every row, as the full-row Metropolis sweep does (ising_fused_rows.hip);
// at step i it runs four updates, each a row behind the one it needs:
//   a0[i+1]  first colour of sweep 1, from the old rows i .. i+2 of the second
//   a1[i]    second colour of sweep 1, from a0[i-1 .. i+1]
//   b0[i-1]  first colour of sweep 2, from a1[i-2 .. i]
//   b1[i-2]  second colour of sweep 2, from b0[i-3 .. i-1]
// The rows a band needs from its neighbours' bands are updated again (four
// rows above it, three below; the draws being none and every site's demon
// read from the old buffers, both copies agree): R + 8 steps for R rows. The
// demons between the two sweeps wait two steps in LDS, where each lane reads
// back its own words. The words beside a wave's columns come through LDS, one
// barrier a step.
//
// Rows of any number of words: lanes past the last word follow the next row
// (their loads are bounded by the buffer, nothing of theirs is stored or
// counted) and the word after the last is replaced by word 0 where its left
// neighbour reads it. Reversed sweeps exchange the colours: the host swaps
// the planes, REV the same-row sides.
//
// One MI355X, us a sweep, against one sweep a launch (forward) or two passes
// in place (reversed, and sides the wave tiles do not cover): 4104^2 16.9 (two
// passes 20.9), 6144^2 19.9 (37.2), 8192^2 30.7 (65.0; reversed 30.7 against
// 55.1), 10000^2 54.7 (81.9), 16384^2 106.7 (249.5; reversed 105.8 against
// 292.2): 2516 site updates/ns, 5.3 TB/s and two thirds of the vector rate;
// 32768^2 441.8 (839.1).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_creutz.hpp"
#include "ising_creutz_pairs.hpp"
#include "ising_device.hpp"
#include "ising_fused_core.hpp"

namespace ising {

namespace {

constexpr uint32_t kMaxWaves = 16;
constexpr int kHaloSteps = 8;

__device__ __forceinline__ void lds_only_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t bounded_rsrc(const uint32_t* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p), 0, bytes, 0x00020000);
}

// Update of one lane's CW words of a row: spins own, demons dem (in place),
// the other colour's rows above, below and alongside, and the words beside
// the wave's columns (left for P == 0, right for P == 1).
template <int CW, int P, bool OBS>
__device__ __forceinline__ Row<CW> creutz_update(const Row<CW>& own, Row<CW>& dem, const Row<CW>& up,
                                                 const Row<CW>& dn, const Row<CW>& same, uint32_t edge,
                                                 const uint32_t (&keep)[CW], uint32_t& sad) {
    const uint32_t nb = P ? from_right(same.v[0], edge) : from_left(same.v[CW - 1], edge);
    Row<CW> out;
#pragma unroll
    for (int w = 0; w < CW; ++w) {
        uint32_t S;
        if (P) S = __builtin_amdgcn_alignbyte(w + 1 < CW ? same.v[w + 1 < CW ? w + 1 : 0] : nb, same.v[w], 1);
        else S = __builtin_amdgcn_alignbyte(same.v[w], w > 0 ? same.v[w > 0 ? w - 1 : 0] : nb, 3);
        const uint32_t n = up.v[w] + dn.v[w] + same.v[w] + S;
        creutz_word(own.v[w], n, dem.v[w], out.v[w], dem.v[w]);
        if (OBS) sad = __builtin_amdgcn_sad_u8((out.v[w] << 2) & keep[w], n & keep[w], sad);
    }
    return out;
}

template <int CW, bool REV, bool RAGGED>
__global__ __launch_bounds__(1024) void k_creutz_pairs(CreutzPairArgs a) {
    extern __shared__ uint32_t held[];  // demons between the sweeps: [colour][2 rows][lane-major words]
    __shared__ uint32_t pub[2][kMaxWaves][8];  // [buffer][wave][c1, a0, a1, b0][first, last]
    __shared__ int64_t wpart[kMaxWaves][4];
    const uint32_t band = xcd_block(gridDim.x);
    const uint32_t lane = threadIdx.x & 63u, nw = blockDim.x >> 6;
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t wl = w == 0u ? nw - 1u : w - 1u, wr = w + 1u == nw ? 0u : w + 1u;
    const uint32_t L = a.L, Hw = a.Hw;
    const int R = (int)a.rows, r0 = (int)(band * a.rows), r1 = min(r0 + R, (int)L);  // rows r0 .. r1 - 1
    const uint32_t x = w * 64u * CW + lane * CW, xb = x * 4u;
    const uint32_t plane_bytes = L * Hw * 4u;
    const __amdgpu_buffer_rsrc_t rs0 = bounded_rsrc(a.s0, plane_bytes), rs1 = bounded_rsrc(a.s1, plane_bytes);
    const __amdgpu_buffer_rsrc_t rm0 = bounded_rsrc(a.m0, plane_bytes), rm1 = bounded_rsrc(a.m1, plane_bytes);
    const __amdgpu_buffer_rsrc_t ws0 = bounded_rsrc(a.d0, plane_bytes), ws1 = bounded_rsrc(a.d1, plane_bytes);
    const __amdgpu_buffer_rsrc_t wm0 = bounded_rsrc(a.e0, plane_bytes), wm1 = bounded_rsrc(a.e1, plane_bytes);
    auto rbyte = [&](int i) { return wrap_row(i, L) * Hw * 4u; };

    // the lane's words of the row (keep: all ones) and, ragged, the word that
    // stands for word 0 after the last one
    uint32_t keep[CW];
    uint32_t ghost[CW];
    uint32_t words = 0;
#pragma unroll
    for (int v = 0; v < CW; ++v) {
        const bool in = !RAGGED || x + (uint32_t)v < Hw;
        keep[v] = in ? ~0u : 0u;
        words += in ? 1u : 0u;
        ghost[v] = RAGGED && x + (uint32_t)v == Hw ? ~0u : 0u;
    }
    const uint32_t end = Hw - 1u;  // the row's last word: its wave, lane and place in the lane
    const uint32_t end_lane = RAGGED && w + 1u == nw ? (end % (64u * CW)) / CW : 63u;
    const uint32_t end_v = RAGGED && w + 1u == nw ? end % CW : CW - 1u;
    uint32_t is_end[CW];
#pragma unroll
    for (int v = 0; v < CW; ++v) is_end[v] = end_v == (uint32_t)v ? ~0u : 0u;
    auto put_ends = [&](uint32_t buf, uint32_t f, const Row<CW>& r) {
        if (lane == 0u) pub[buf][w][2u * f] = r.v[0];
        if (lane == end_lane) {
            uint32_t v = 0;
#pragma unroll
            for (int k = 0; k < CW; ++k) v |= RAGGED ? r.v[k] & is_end[k] : (k == CW - 1 ? r.v[k] : 0u);
            pub[buf][w][2u * f + 1u] = v;
        }
    };
    auto beside = [&](uint32_t buf, int P, uint32_t f) { return P ? pub[buf][wr][2u * f] : pub[buf][wl][2u * f + 1u]; };
    // Ragged, right neighbours: word 0 in the place after the row's last word
    auto closed = [&](const Row<CW>& r, int P, uint32_t edge) {
        Row<CW> o;
#pragma unroll
        for (int k = 0; k < CW; ++k) o.v[k] = RAGGED && P ? r.v[k] ^ ((r.v[k] ^ edge) & ghost[k]) : r.v[k];
        return o;
    };
    auto store = [&](__amdgpu_buffer_rsrc_t rs, int i, const Row<CW>& r) {
        const uint32_t off = xb + (uint32_t)i * Hw * 4u;
        if (!RAGGED || words == CW) {
            st<CW>(rs, off, r);
        } else {
#pragma unroll
            for (int k = 0; k < CW; ++k)
                if (keep[k]) __builtin_amdgcn_raw_buffer_store_b32(r.v[k], rs, off + 4u * (uint32_t)k, 0, kRowCachePolicy);
        }
    };
    uint32_t* const mine = held + w * 64u * CW + lane;
    const uint32_t row_words = nw * 64u * CW;
    auto hold = [&](uint32_t colour, uint32_t k, const Row<CW>& r) {
#pragma unroll
        for (int v = 0; v < CW; ++v) mine[(colour * 2u + k) * row_words + (uint32_t)v * 64u] = r.v[v];
    };
    auto held_row = [&](uint32_t colour, uint32_t k) {
        Row<CW> r;
#pragma unroll
        for (int v = 0; v < CW; ++v) r.v[v] = mine[(colour * 2u + k) * row_words + (uint32_t)v * 64u];
        return r;
    };

    // rings, indexed by (row - (r0 - 4)) & 3 (or & 1): old rows of the second
    // colour, of the first, their demons; sweep 1; sweep 2's first colour
    Row<CW> c1[4], c0[2], m0[2], m1[2], a0[4] = {}, a1[4] = {}, b0[4] = {};
    const int i0 = r0 - 4;
    c1[0] = ld<CW>(rs1, xb, rbyte(i0));
    c1[1] = ld<CW>(rs1, xb, rbyte(i0 + 1));
    c1[2] = ld<CW>(rs1, xb, rbyte(i0 + 2));
    c0[1] = ld<CW>(rs0, xb, rbyte(i0 + 1));
    m0[1] = ld<CW>(rm0, xb, rbyte(i0 + 1));
    m1[0] = ld<CW>(rm1, xb, rbyte(i0));
    if (threadIdx.x < 2u * kMaxWaves * 8u) (&pub[0][0][0])[threadIdx.x] = 0u;
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) hold(k >> 1, k & 1u, a0[0]);
    __syncthreads();
    put_ends(0u, 0u, c1[1]);
    lds_only_barrier();
    uint32_t sad1 = 0, sad2 = 0, ups1 = 0, ups2 = 0, dummy = 0;

#pragma unroll 1
    for (int k = 0; k < R + kHaloSteps; k += 4) {
        uint32_t up1 = 0, up2 = 0;  // bytewise
        auto step = [&](auto uc) {
            constexpr int u = decltype(uc)::value;
            constexpr uint32_t rd = u & 1, wrb = rd ^ 1u;
            constexpr int P = ((u & 1) == 0) != REV ? 1 : 0;  // the same for the four rows: they alternate with the colours
            const int i = i0 + k + u;
            // the next step's rows
            c1[(u + 3) & 3] = ld<CW>(rs1, xb, rbyte(i + 3));
            c0[u & 1] = ld<CW>(rs0, xb, rbyte(i + 2));
            m0[u & 1] = ld<CW>(rm0, xb, rbyte(i + 2));
            m1[(u + 1) & 1] = ld<CW>(rm1, xb, rbyte(i + 1));
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t g0 = beside(rd, P, 0u), g1 = beside(rd, P, 1u), g2 = beside(rd, P, 2u), g3 = beside(rd, P, 3u);
            // sweep 1
            Row<CW> dm0 = m0[(u + 1) & 1], dm1 = m1[u & 1];
            a0[(u + 1) & 3] = creutz_update<CW, P, false>(c0[(u + 1) & 1], dm0, c1[u & 3], c1[(u + 2) & 3],
                                                          closed(c1[(u + 1) & 3], P, g0), g0, keep, dummy);
            uint32_t sad = 0;
            a1[u & 3] = creutz_update<CW, P, true>(c1[u & 3], dm1, a0[(u + 3) & 3], a0[(u + 1) & 3],
                                                   closed(a0[u & 3], P, g1), g1, keep, sad);
            if (i >= r0 && i < r1) {
                sad1 += sad;
#pragma unroll
                for (int v = 0; v < CW; ++v) up1 += (a1[u & 3].v[v] + a0[u & 3].v[v]) & keep[v];
            }
            // sweep 2, with the demons of two steps ago
            Row<CW> em0 = held_row(0u, (u + 1) & 1u), em1 = held_row(1u, u & 1u);
            hold(0u, (u + 1) & 1u, dm0);
            hold(1u, u & 1u, dm1);
            b0[(u + 3) & 3] = creutz_update<CW, P, false>(a0[(u + 3) & 3], em0, a1[(u + 2) & 3], a1[u & 3],
                                                          closed(a1[(u + 3) & 3], P, g2), g2, keep, dummy);
            if (i - 1 >= r0 && i - 1 < r1) {
                store(ws0, i - 1, b0[(u + 3) & 3]);
                store(wm0, i - 1, em0);
            }
            sad = 0;
            const Row<CW> b1 = creutz_update<CW, P, true>(a1[(u + 2) & 3], em1, b0[(u + 1) & 3], b0[(u + 3) & 3],
                                                          closed(b0[(u + 2) & 3], P, g3), g3, keep, sad);
            if (i - 2 >= r0 && i - 2 < r1) {
                store(ws1, i - 2, b1);
                store(wm1, i - 2, em1);
                sad2 += sad;
#pragma unroll
                for (int v = 0; v < CW; ++v) up2 += (b1.v[v] + b0[(u + 2) & 3].v[v]) & keep[v];
            }
            // for the next step
            put_ends(wrb, 0u, c1[(u + 2) & 3]);
            put_ends(wrb, 1u, a0[(u + 1) & 3]);
            put_ends(wrb, 2u, a1[u & 3]);
            put_ends(wrb, 3u, b0[(u + 3) & 3]);
            lds_only_barrier();
            __builtin_amdgcn_sched_barrier(0);
        };
        step(Step<0>{});
        step(Step<1>{});
        step(Step<2>{});
        step(Step<3>{});
        ups1 = __builtin_amdgcn_sad_u8(up1, 0u, ups1);  // at most 8 CW a byte
        ups2 = __builtin_amdgcn_sad_u8(up2, 0u, ups2);
    }

    // (B, M) of both sweeps: B = 16 words - 2 sad, M = 2 ups - 8 words
    const int64_t n = (int64_t)words * (r1 - r0);
    int64_t v[4] = {16 * n - 2 * (int64_t)sad1, 2 * (int64_t)ups1 - 8 * n, 16 * n - 2 * (int64_t)sad2,
                    2 * (int64_t)ups2 - 8 * n};
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = wave_sum_i64(v[k]);
    if (lane == 0u)
#pragma unroll
        for (int k = 0; k < 4; ++k) wpart[w][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 4u) {
        int64_t s = 0;
        for (uint32_t q = 0; q < nw; ++q) s += wpart[q][threadIdx.x];
        const uint32_t sweep = threadIdx.x >> 1;
        a.part[2u * ((size_t)sweep * gridDim.x + band) + (threadIdx.x & 1u)] = s;
    }
}

template <int CW, bool REV>
const void* kernel_of(bool ragged) {
    return ragged ? reinterpret_cast<const void*>(&k_creutz_pairs<CW, REV, true>)
                  : reinterpret_cast<const void*>(&k_creutz_pairs<CW, REV, false>);
}

}  // namespace

// The fewest words a lane whose waves span the row: 4096-word rows need four
// (125 registers, one workgroup of 16 waves a compute unit).
bool creutz_pairs_shape(uint32_t L, uint32_t cus, CreutzPairShape* out) {
    if (L % 8u != 0u || L < 64u || cus == 0u) return false;
    const uint32_t Hw = L / 8u;
    uint32_t cw = 1u;
    while (cw <= 4u && (Hw + 64u * cw - 1u) / (64u * cw) > kMaxWaves) cw *= 2u;
    if (cw > 4u) return false;
    const uint32_t waves = (Hw + 64u * cw - 1u) / (64u * cw);
    // one workgroup a compute unit, but bands of at least 16 rows (eight more
    // steps than rows)
    uint32_t rows = ((L + cus - 1u) / cus + 3u) / 4u * 4u;
    if (rows < 16u) rows = 16u;
    *out = CreutzPairShape{cw, waves * 64u, rows, (L + rows - 1u) / rows, 16u * waves * 64u * cw, Hw % (64u * cw) != 0u};
    return true;
}

hipError_t launch_creutz_pair(const CreutzPairArgs& a, const CreutzPairShape& s, bool reverse, hipStream_t stream) {
    const void* k = s.cw == 1u ? (reverse ? kernel_of<1, true>(s.ragged) : kernel_of<1, false>(s.ragged))
                    : s.cw == 2u ? (reverse ? kernel_of<2, true>(s.ragged) : kernel_of<2, false>(s.ragged))
                                 : (reverse ? kernel_of<4, true>(s.ragged) : kernel_of<4, false>(s.ragged));
    if (s.lds > 49152u) {  // with the kernel's own LDS beyond the default limit
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)s.lds);
        if (e != hipSuccess) return e;
    }
    CreutzPairArgs arg = a;
    arg.rows = s.rows;
    void* args[] = {&arg};
    return hipLaunchKernel(k, dim3(s.bands), dim3(s.threads), args, s.lds, stream);
}

}  // namespace ising
