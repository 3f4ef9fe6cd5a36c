// One sweep a launch over wave tiles, for rows of any number of words: large
// lattices read once and written once a sweep (2 bytes a site update).
//
// The walk down a tile is k_fused's (ising_fused.hip): a wave holds 64 CW
// words of a row and updates colour 0 of row i + 1 and colour 1 of row i, the
// words beside the tile computed up front, one lane a row. That kernel takes
// rows of whole tiles only. Here the last column may end anywhere: its waves
// run a variant that puts the word beside the tile after the row's last word
// and masks stores and sums (the branch is uniform over a wave, so the other
// columns run the plain update), and a lattice's last band may have fewer
// rows.
//
// Bound by the vector units: two sweeps a launch by full-row workgroups, at
// half the traffic, measured no faster (20000^2 259 us a sweep against 225,
// 32760^2 514 and 525). Us a sweep on one MI355X,
// before and now: lattices in a field, whose band update by bits costs half as
// much again as without, 4104^2 27.2 and 19.5, 8192^2 51.0 and 46.2, 10000^2
// 88.2 and 70.8 (and, without the nontemporal hint where the buffers stay in
// cache, 18.1, 37.8 and 58.2), 12296^2 145 and 99, 16384^2 182 and 156; sides beyond the
// bands, by two passes, 16392^2 216 and 177, 18000^2 239 and 190, 20000^2 264
// and 225, 26008^2 545 and 350, 32760^2 856 and 525 (2042 site updates/ns, 4.1
// TB/s). Whole columns only (sides of 512) stay with k_fused, 5% faster for
// its fixed tile height (29696^2 398 and 427).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_device.hpp"
#include "ising_fused_core.hpp"
#include "ising_tiles.hpp"

namespace ising {

namespace {

constexpr uint32_t kThreads = 256;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t bounded_rsrc(const uint32_t* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p), 0, bytes, 0x00020000);
}

// The words of a tile's rows that the lane holds.
template <int CW>
struct Part {
    uint32_t words;      // 0 .. CW
    uint32_t keep[CW];   // all ones: a word of the row
    uint32_t after[CW];  // all ones: the place after the row's last word
    bool last;           // the lane whose last word is the row's last
};

// update_row (ising_fused_core.hpp) for a tile that ends before its last
// lane's last word: the word after the row's last is `edge`, and only the
// row's words count.
template <int CW, int P, bool OBS>
__device__ __forceinline__ Row<CW> update_part(const LdsTable& lt, const Part<CW>& pt, const Row<CW>& own,
                                               const Row<CW>& up, const Row<CW>& dn, const Row<CW>& same, uint32_t edge,
                                               const Row<CW>& xw, uint32_t rowoff, uint32_t t, uint32_t c, uint32_t k0,
                                               uint32_t k1, uint32_t& sad) {
    Row<CW> al = same;
#pragma unroll
    for (int w = 0; w < CW; ++w)
        if (P) al.v[w] = (same.v[w] & ~pt.after[w]) | (edge & pt.after[w]);
    uint32_t nb = P ? from_right(al.v[0], edge) : from_left(al.v[CW - 1], edge);
    if (P && pt.last) nb = edge;
    Row<CW> out;
#pragma unroll
    for (int w = 0; w < CW; ++w) {
        uint32_t S;
        if (P) S = __builtin_amdgcn_alignbyte(w + 1 < CW ? al.v[w + 1 < CW ? w + 1 : 0] : nb, al.v[w], 1);
        else S = __builtin_amdgcn_alignbyte(al.v[w], w > 0 ? al.v[w > 0 ? w - 1 : 0] : nb, 3);
        const uint32_t n = (up.v[w] + dn.v[w] + S) + al.v[w];
        const uint64_t p0 = mad_u64_uniform(xw.v[0], kPhiloxM0, (uint64_t)kPhiloxM0 * (rowoff + (uint32_t)w));
        const AcceptEntries ent = accept_entries(lt, (own.v[w] << 3) + n);
        __builtin_amdgcn_sched_barrier(0);
        out.v[w] = accept_from(ent, philox_p0(p0, t, c, 0u, k0, k1));
        if (OBS) sad = sad_misaligned(out.v[w] & pt.keep[w], n & pt.keep[w], sad);
    }
    return out;
}

// One tile: R rows from r0, the columns from word X0 (PART: `wds` words of
// them, fewer than 64 CW). The rows are those of k_fused (ising_fused.hip).
template <int CW, bool PART, int POLICY>
__device__ __forceinline__ void walk(const LdsTable& lt, const FusedArgs& a, uint32_t X0, uint32_t wds, int r0, int R,
                                     int64_t* out) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t L = a.L, Hw = a.Hw, t = a.t, k0 = a.k0, k1 = a.k1;
    Part<CW> pt;
    pt.words = CW;
    pt.last = false;
    uint32_t x = X0 + lane * CW;
    if (PART) {
        const uint32_t at = lane * CW;
        pt.words = at >= wds ? 0u : min(wds - at, (uint32_t)CW);
        pt.last = at + CW == wds;
#pragma unroll
        for (int v = 0; v < CW; ++v) {
            pt.keep[v] = at + (uint32_t)v < wds ? ~0u : 0u;
            pt.after[v] = at + (uint32_t)v == wds ? ~0u : 0u;
        }
        if (at >= wds) x = X0 + (wds - 1u) / CW * CW;  // idle lanes follow the last one
    }
    const uint32_t xl = X0 == 0 ? Hw - 1 : X0 - 1;
    const uint32_t xr = X0 + wds == Hw ? 0u : X0 + wds;
    const uint32_t* __restrict__ s0 = a.src0;
    const uint32_t* __restrict__ s1 = a.src1;
    auto row_ptr = [&](const uint32_t* base, int i) { return base + (size_t)wrap_row(i, L) * Hw; };

    // lane l: the old colour-1 word just outside the tile that row r0 + 1 +
    // l's colour-0 update needs, and the new colour-0 word just outside it
    // that row r0 + l's colour-1 update needs
    uint32_t edge_c1 = 0, edge_c0 = 0;
    if (lane < (uint32_t)R) {
        const int j = r0 + 1 + (int)lane;
        const uint32_t rj = wrap_row(j, L);
        edge_c1 = row_ptr(s1, j)[(rj & 1u) ? xr : xl];
        const int i = r0 + (int)lane;
        const uint32_t ri = wrap_row(i, L);
        const uint32_t xe = (ri & 1u) ? xl : xr;
        const uint32_t pe = ri & 1u;
        const uint32_t xn = pe ? (xe + 1 == Hw ? 0u : xe + 1) : (xe == 0 ? Hw - 1 : xe - 1);
        const uint32_t own = row_ptr(s0, i)[xe];
        const uint32_t up = row_ptr(s1, i - 1)[xe];
        const uint32_t dn = row_ptr(s1, i + 1)[xe];
        const uint32_t same = row_ptr(s1, i)[xe];
        const uint32_t nbw = row_ptr(s1, i)[xn];
        const uint32_t S = pe ? __builtin_amdgcn_alignbyte(nbw, same, 1) : __builtin_amdgcn_alignbyte(same, nbw, 3);
        const uint32_t n = up + dn + same + S;
        edge_c0 = accept_word(lt, (own << 3) + n, philox(ri * Hw + xe, t, 0u, 0u, k0, k1));
    }

    uint32_t sad = 0, ups = 0, ups8 = 0, dummy = 0;
    const uint32_t xb = x * 4u;
    Row<CW> xw;
#pragma unroll
    for (int w = 0; w < CW; ++w) xw.v[w] = x + (uint32_t)w;
    const uint32_t bytes = L * Hw * 4u;  // loads past a plane's end (a part of the last row's last words) are 0
    const __amdgpu_buffer_rsrc_t rs0 = bounded_rsrc(s0, bytes), rs1 = bounded_rsrc(s1, bytes);
    const __amdgpu_buffer_rsrc_t rd0 = bounded_rsrc(a.dst0, bytes), rd1 = bounded_rsrc(a.dst1, bytes);
    auto rword = [&](int i) { return wrap_row(i, L) * Hw; };
    auto rbyte = [&](int i) { return rword(i) * 4u; };
    auto store = [&](__amdgpu_buffer_rsrc_t rs, uint32_t off, const Row<CW>& r) {
        if (!PART || pt.words == CW) {
            st<CW, POLICY>(rs, off, r);
        } else {
#pragma unroll
            for (int v = 0; v < CW; ++v)
                if (pt.keep[v]) __builtin_amdgcn_raw_buffer_store_b32(r.v[v], rs, off + 4u * (uint32_t)v, 0, POLICY);
        }
    };
    // colour 0 of a row (not counted) and colour 1 (counted)
    auto first = [&](auto pc, const Row<CW>& own, const Row<CW>& up, const Row<CW>& dn, const Row<CW>& same,
                     uint32_t edge, uint32_t rowoff) {
        constexpr int P = decltype(pc)::value;
        if constexpr (PART)
            return update_part<CW, P, false>(lt, pt, own, up, dn, same, edge, xw, rowoff, t, 0u, k0, k1, dummy);
        else
            return update_row<CW, P, false>(lt, own, up, dn, same, edge, xw, rowoff, t, 0u, k0, k1, dummy);
    };
    auto second = [&](auto pc, const Row<CW>& own, const Row<CW>& up, const Row<CW>& dn, const Row<CW>& same,
                      uint32_t edge, uint32_t rowoff) {
        constexpr int P = decltype(pc)::value;
        if constexpr (PART)
            return update_part<CW, P, true>(lt, pt, own, up, dn, same, edge, xw, rowoff, t, 1u, k0, k1, sad);
        else
            return update_row<CW, P, true>(lt, own, up, dn, same, edge, xw, rowoff, t, 1u, k0, k1, sad);
    };

    // rings: c1[(row - r0) & 3] old colour-1 rows, c0o[(row - r0) & 1] old
    // colour-0 rows, c0n[(row - r0 + 1) & 3] new colour-0 rows
    Row<CW> c1[4], c0o[2], c0n[4];
    const Row<CW> c1m2 = ld<CW, POLICY>(rs1, xb, rbyte(r0 - 2));
    const Row<CW> c1m1 = ld<CW, POLICY>(rs1, xb, rbyte(r0 - 1));
    c1[0] = ld<CW, POLICY>(rs1, xb, rbyte(r0));
    c1[1] = ld<CW, POLICY>(rs1, xb, rbyte(r0 + 1));
    c1[2] = ld<CW, POLICY>(rs1, xb, rbyte(r0 + 2));
    const Row<CW> c0om1 = ld<CW, POLICY>(rs0, xb, rbyte(r0 - 1));
    c0o[0] = ld<CW, POLICY>(rs0, xb, rbyte(r0));
    c0o[1] = ld<CW, POLICY>(rs0, xb, rbyte(r0 + 1));
    const uint32_t eR = row_ptr(s1, r0 - 1)[xr];
    const uint32_t eL = row_ptr(s1, r0)[xl];
    c0n[0] = first(Step<1>{}, c0om1, c1m2, c1[0], c1m1, eR, rword(r0 - 1));
    c0n[1] = first(Step<0>{}, c0o[0], c1m1, c1[1], c1[0], eL, rword(r0));
    store(rd0, xb + rbyte(r0), c0n[1]);

#pragma unroll 1
    for (int k = 0; k < R; k += 4) {
        auto step = [&](auto uc) {
            constexpr int u = decltype(uc)::value;
            const int i = r0 + k + u;
            c1[(u + 3) & 3] = ld<CW, POLICY>(rs1, xb, rbyte(i + 3));
            c0o[u & 1] = ld<CW, POLICY>(rs0, xb, rbyte(i + 2));
            const uint32_t e1 = (uint32_t)__builtin_amdgcn_readlane((int)edge_c1, k + u);
            const uint32_t e0 = (uint32_t)__builtin_amdgcn_readlane((int)edge_c0, k + u);
            using P = Step<(u & 1) == 0 ? 1 : 0>;
            c0n[(u + 2) & 3] = first(P{}, c0o[(u + 1) & 1], c1[u & 3], c1[(u + 2) & 3], c1[(u + 1) & 3], e1, rword(i + 1));
            const Row<CW> c1n =
                second(P{}, c1[u & 3], c0n[u & 3], c0n[(u + 2) & 3], c0n[(u + 1) & 3], e0, rword(i));
            if (k + u + 1 < R) store(rd0, xb + rbyte(i + 1), c0n[(u + 2) & 3]);
            store(rd1, xb + rbyte(i), c1n);
#pragma unroll
            for (int w = 0; w < CW; ++w) {
                const uint32_t both = c1n.v[w] + c0n[(u + 1) & 3].v[w];
                ups8 += PART ? both & pt.keep[w] : both;  // at most 8 CW a byte over the four steps
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        step(Step<0>{});
        step(Step<1>{});
        step(Step<2>{});
        step(Step<3>{});
        ups = __builtin_amdgcn_sad_u8(ups8, 0u, ups);
        ups8 = 0;
    }

    // B = 16 words - 2 sad, M = 2 ups - 8 words
    const int64_t words = (int64_t)R * pt.words;
    int64_t b = 16 * words - 2 * (int64_t)sad;
    int64_t m = 2 * (int64_t)ups - 8 * words;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        b += __shfl_xor(b, off, 64);
        m += __shfl_xor(m, off, 64);
    }
    if (lane == 0) {
        out[0] = b;
        out[1] = m;
    }
}

// At least four waves per SIMD (at most 128 registers).
template <int CW, int POLICY>
__global__ void __launch_bounds__(kThreads, 4) k_tiles(FusedArgs a, AcceptTable at, PartialReduce red, uint32_t rows) {
    __shared__ LdsTable lt;
    load_table(lt, at);
    __syncthreads();
    const uint32_t block = xcd_block(gridDim.x);
    if (block == 0) reduce_partials(red);
    const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)(block * (kThreads / 64u) + (threadIdx.x >> 6)));
    if (tile >= a.n_tiles) return;  // whole wave
    const uint32_t tx = tile % a.n_tx, ty = tile / a.n_tx;
    const uint32_t X0 = tx * 64u * CW, wds = min(64u * CW, a.Hw - X0);
    const int r0 = (int)(ty * rows), R = (int)min(rows, a.L - ty * rows);  // a multiple of 4: L % 8 == 0
    int64_t* const out = a.part + 2ull * tile;
    if (wds == 64u * CW) walk<CW, false, POLICY>(lt, a, X0, wds, r0, R, out);
    else walk<CW, true, POLICY>(lt, a, X0, wds, r0, R, out);
}

}  // namespace

// Us a sweep by words a lane / rows a tile: 6144^2 29.2 with 2/8, 32.8 2/16,
// 31.6 4/8; 8192^2 50.0, 46.2, 43.9; 14000^2 122, 118, 123 (4/16 119);
// 20000^2 227 with 2/16, 225 4/16, 227 4/32; 32760^2 554, 525, 573. One word a
// lane is slower everywhere (10000^2 73 at best against 68), 64 rows leave too
// few waves.
bool tiles_shape(uint32_t L, TileShape* out) {
    if (L % 8u != 0u || L < 64u) return false;
    const uint32_t Hw = L / 8u;
    const uint32_t cw = L <= 16384u ? 2u : 4u, rows = L < 8192u ? 8u : 16u;
    const uint32_t n_tx = (Hw + 64u * cw - 1u) / (64u * cw);
    *out = TileShape{cw, rows, n_tx, n_tx * ((L + rows - 1u) / rows)};
    return true;
}

hipError_t launch_tiles(const FusedArgs& a, const AcceptTable& at, const TileShape& shape, const PartialReduce& red,
                        hipStream_t s) {
    // whole groups of eight blocks, one for each chiplet (xcd_block)
    const uint32_t blocks = (shape.tiles + 8u * (kThreads / 64u) - 1u) / (8u * (kThreads / 64u)) * 8u;
    const auto kernel = shape.cw != 2u                          ? k_tiles<4, kRowCachePolicy>
                        : rows_stay_cached((uint64_t)a.L * a.L) ? k_tiles<2, kRowCachePlain>
                                                                : k_tiles<2, kRowCachePolicy>;
    kernel<<<blocks, kThreads, 0, s>>>(a, at, red, shape.rows);
    return hipGetLastError();
}

}  // namespace ising
