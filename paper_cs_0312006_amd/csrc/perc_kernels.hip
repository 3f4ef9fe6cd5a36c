// HIP kernels of the gfx950 site-percolation engine (Section 2.3 of Tomov
// et al. 2003): porosity draw, then invasion of the medium from the source.
//
// The paper's GPU program spreads the cluster by one pass over the whole
// lattice per invasion step, so a medium whose cluster needs D steps costs
// D full passes. Here a launch advances the invasion by 32 passes at once,
// and only where the front is: pores and invaded sites are kept as bit maps
// of 64 x 64 tiles, and a wave takes one tile with the 32 sites around it on
// every side (128 x 128 sites, two rows of 128 bits a lane), runs 32 passes
// of the invasion on the bits and writes back the tile's own 64 x 64. A pass
// moves the front by one site, so what lies outside the 128 x 128 cannot
// reach the tile within the launch: every tile ends with exactly the sites
// invaded by that pass, whatever the order of the tiles, and each site's
// arrival pass is written once. A tile is listed for the next launch only
// where the last pass left new sites in its 128 x 128.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_device.hpp"
#include "perc_launch.hpp"

namespace perc {

namespace {

// DPP controls (GFX9): whole-wave shift by one lane; zero enters at the end.
constexpr int kDppWaveShl1 = 0x130;  // lane l reads lane l+1
constexpr int kDppWaveShr1 = 0x138;  // lane l reads lane l-1

__device__ __forceinline__ uint32_t prev_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppWaveShr1, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t next_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppWaveShl1, 0xf, 0xf, true);
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor(v, off, 64));
    return v;
}

// Four dwords of a row of 128 sites: 32 left of the tile, its 64, 32 right.
struct Row128 {
    uint32_t v[4];
};

// The row's sites x and the pores next to them in the row itself and to
// `own` and `other`, the rows above and below.
__device__ __forceinline__ Row128 spread(const Row128& x, const Row128& own, const Row128& other, const Row128& pores) {
    Row128 r;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t before = __builtin_amdgcn_alignbit(x.v[k], k > 0 ? x.v[k > 0 ? k - 1 : 0] : 0u, 31);
        const uint32_t after = __builtin_amdgcn_alignbit(k < 3 ? x.v[k < 3 ? k + 1 : 0] : 0u, x.v[k], 1);
        r.v[k] = (((before | after | own.v[k]) | other.v[k]) & pores.v[k]) | x.v[k];
    }
    return r;
}

}  // namespace

// Porosity draw (a site is a pore iff its 32-bit draw is below pthr; four
// consecutive row-major sites share a Philox call), the pore bytes and bit
// map, and the state before the first pass: the source's pores invaded at
// pass 0, every other arrival -1. A wave takes 256 sites of one row, four a
// lane; where the row does not start a call a lane's four sites take words
// of two calls. Blocks of y = m work on medium m.
__global__ void __launch_bounds__(kThreads) k_perc_draw(const Medium* __restrict__ media, WorkLists w, Result* res) {
    const Medium& md = media[blockIdx.y];
    const uint32_t L = md.L, n_tx = md.n_tx, n_tiles = n_tx * md.n_ty;
    const uint32_t tid = blockIdx.x * kThreads + threadIdx.x, threads = gridDim.x * kThreads;
    if (blockIdx.y == 0)
        for (uint32_t k = tid; k < 3u * kSubs; k += threads) w.len[k] = 0u;
    for (uint32_t t = tid; t < n_tiles; t += threads) {
        md.queued[0][t] = 0u;
        md.queued[1][t] = 0u;
        md.stat[t] = TileStat{0u, 0u, 0u, 0u};
    }
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t segs = (L + 255u) / 256u, rows = md.n_ty * kTile;  // rows past the lattice: empty map
    const uint64_t chunks = (uint64_t)rows * segs, waves = threads >> 6;
    uint32_t* const pmap = reinterpret_cast<uint32_t*>(md.pmap);
    uint32_t* const reach0 = reinterpret_cast<uint32_t*>(md.reach[0]);
    uint32_t* const reach1 = reinterpret_cast<uint32_t*>(md.reach[1]);
    uint32_t cnt = 0;
    for (uint64_t ch = (uint64_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6)); ch < chunks; ch += waves) {
        const uint32_t i = (uint32_t)(ch / segs), sg = (uint32_t)(ch - (uint64_t)i * segs);
        const uint32_t j = sg * 256u + 4u * lane;
        const uint32_t nv = (i < L && j < L) ? min(4u, L - j) : 0u;
        const uint64_t ord = (uint64_t)i * L + j;
        const uint32_t o = (uint32_t)((uint64_t)i * L) & 3u;
        uint32_t nib = 0, src = 0;
        if (i < L) {  // the whole wave
            const uint32_t q = (uint32_t)(ord >> 2);
            const uint4 r = ising::philox(q, 0u, 0u, 2u, md.k0, md.k1);
            uint32_t u[4] = {r.x, r.y, r.z, r.w};
            if (o) {  // words o .. 3 of this call, 0 .. o - 1 of the next
                const uint4 n = ising::philox(q + 1u, 0u, 0u, 2u, md.k0, md.k1);
                if (o == 1u) u[0] = r.y, u[1] = r.z, u[2] = r.w, u[3] = n.x;
                else if (o == 2u) u[0] = r.z, u[1] = r.w, u[2] = n.x, u[3] = n.y;
                else u[0] = r.w, u[1] = n.x, u[2] = n.y, u[3] = n.z;
            }
#pragma unroll
            for (uint32_t b = 0; b < 4u; ++b) {
                const bool p = b < nv && (uint64_t)u[b] < md.pthr;
                const bool s = md.source == 0u ? i == 0u : (i == md.i0 && j + b == md.j0);
                nib |= (uint32_t)p << b;
                src |= (uint32_t)(p && s) << b;
            }
            const uint32_t bytes = (nib & 1u) | (nib & 2u) << 7 | (nib & 4u) << 14 | (nib & 8u) << 21;
            const uint4 a = make_uint4(src & 1u ? 0u : ~0u, src & 2u ? 0u : ~0u, src & 4u ? 0u : ~0u, src & 8u ? 0u : ~0u);
            if (nv == 4u && o == 0u) {  // both arrays aligned (L % 4 == 0, or every fourth row)
                *reinterpret_cast<uint32_t*>(md.pore + ord) = bytes;
                *reinterpret_cast<uint4*>(md.arr + ord) = a;
            } else {
                const uint32_t av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                for (uint32_t b = 0; b < 4u; ++b)
                    if (b < nv) {
                        md.pore[ord + b] = (uint8_t)(bytes >> (8u * b)) & 1u;
                        md.arr[ord + b] = av[b];
                    }
            }
            cnt += __builtin_popcount(nib);
        }
        // eight lanes' nibbles make a dword of the maps
        uint32_t pw = nib << (4u * (lane & 7u)), sw = src << (4u * (lane & 7u));
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) {
            pw |= (uint32_t)__shfl_xor((int)pw, off, 64);
            sw |= (uint32_t)__shfl_xor((int)sw, off, 64);
        }
        const uint32_t tx = j / kTile;
        if ((lane & 7u) == 0u && tx < n_tx) {
            const size_t k = ((size_t)((i / kTile) * n_tx + tx) * kTile + i % kTile) * 2u + ((j >> 5) & 1u);
            pmap[k] = pw;
            reach0[k] = sw;
            reach1[k] = sw;
        }
    }
    const uint32_t s = ising::wave_sum_u32(cnt);
    __shared__ uint32_t part[kThreads / 64];
    if (lane == 0u) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (uint32_t k = 0; k < kThreads / 64; ++k) t += part[k];
        if (t) atomicAdd(&res[blockIdx.y].pores, t);
    }
}

// Every medium's source tiles, appended to work list 0 (a block a medium):
// the tiles that see a source site within 32 sites.
__global__ void __launch_bounds__(kThreads) k_perc_seed(const Medium* __restrict__ media, WorkLists w) {
    const uint32_t m = blockIdx.x;
    const Medium& md = media[m];
    auto add = [&](uint32_t tx, uint32_t ty) {
        const uint32_t t = ty * md.n_tx + tx, p = list_part(m, tx, ty);
        md.queued[0][t] = 1u;
        w.list[0][(size_t)p * w.cap + atomicAdd(&w.len[p], 1u)] = make_uint2(m, t);
    };
    if (md.source == 0u) {
        for (uint32_t tx = threadIdx.x; tx < md.n_tx; tx += kThreads) add(tx, 0u);
    } else if (threadIdx.x < 9u) {
        const int ty = (int)(md.i0 / kTile) + (int)(threadIdx.x / 3u) - 1;
        const int tx = (int)(md.j0 / kTile) + (int)(threadIdx.x % 3u) - 1;
        if (ty >= 0 && tx >= 0 && ty < (int)md.n_ty && tx < (int)md.n_tx) add((uint32_t)tx, (uint32_t)ty);
    }
}

// Relaxation launch k: passes lo + 1 .. lo + 32 (lo = 32 k), a wave per
// listed tile.
//
// A lane holds rows 2 l and 2 l + 1 of the 128 (rows 32 + 2 l of the tile
// above for lanes 0..15, rows 2 (l - 16) of the tile for 16..47, rows
// 2 (l - 48) of the tile below), so a pass is five operations a dword, the
// neighbour rows being the lane's own or the next lane's (DPP). The pass in
// which each of the tile's sites was invaded is kept bit-sliced: five
// planes, or-ed with the pass's new sites where that bit of the pass number
// is set.
//
// What bounds it: latency, times the launches a run needs (passes / 32). With
// one front tile a SIMD even at 16384^2 nothing hides a launch's 5 us, the
// list entry's 1 us, the maps' 0.6, the 32 passes' 3 (64 operations each) and
// the next list's atomics and the arrivals' stores, 2 together: 14.7 us a
// launch at 16384^2, 12 at 512^2. So the list entry is read beside its count,
// a run of one medium has its descriptor in the kernel arguments, and the
// passes are a loop (unrolled 32 times: 18.6 us a launch at 16384^2). Whole
// runs, against the arrival relaxation of revisited tiles this replaced:
// 512^2 0.82 against 2.0 ms, 2048^2 2.1 against 6.7, 16384^2 17.9 against
// 47.9, 32768^2 42.5 against 125, 48 of 512^2 together 1.1 against 7.4.
template <bool ONE>
__global__ void __launch_bounds__(kRelaxThreads) k_perc_relax(Medium one, const Medium* __restrict__ media,
                                                              WorkLists w, uint32_t pin, uint32_t lin, uint32_t lout,
                                                              uint32_t lclr, uint32_t lo) {
    const uint32_t lane = threadIdx.x;
    if (blockIdx.x == 0u) w.len[lclr * kSubs + lane] = 0u;
    const uint32_t sub = blockIdx.x % kSubs, e0 = blockIdx.x / kSubs, step = gridDim.x / kSubs;
    const uint2* const list = (pin ? w.list[1] : w.list[0]) + (size_t)sub * w.cap;
    uint2* const list_out = pin ? w.list[0] : w.list[1];
    uint2 ent = list[min(e0, w.cap - 1u)];  // beside the count: it is used only if it is there
    const uint32_t n = w.len[lin * kSubs + sub];
    for (uint32_t e = e0; e < n; e += step) {
        if (e != e0) ent = list[e];
        // the entry is the same for the whole wave: keep it scalar
        const uint32_t m = ONE ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane((int)ent.x);
        const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)ent.y);
        const Medium& md = ONE ? one : media[m];
        const uint32_t L = md.L, n_tx = md.n_tx, n_ty = md.n_ty;
        const uint32_t ty = tile / n_tx, tx = tile - ty * n_tx;
        const uint64_t* const rin = pin ? md.reach[1] : md.reach[0];
        uint64_t* const rout = pin ? md.reach[0] : md.reach[1];
        uint32_t* const q_in = pin ? md.queued[1] : md.queued[0];
        uint32_t* const q_out = pin ? md.queued[0] : md.queued[1];
        if (lane == 0u) q_in[tile] = 0u;

        // the lane's two rows of pores and of invaded sites
        const int dy = lane < 16u ? -1 : lane < 48u ? 0 : 1;
        const uint32_t row = 2u * (lane < 16u ? lane + 16u : lane < 48u ? lane - 16u : lane - 48u);
        const int ly = (int)ty + dy;
        const bool y_in = ly >= 0 && ly < (int)n_ty;
        const uint32_t cy = y_in ? (uint32_t)ly : ty;  // clamped: the load stays inside the map
        auto rows_at = [&](const uint64_t* map, int dx, bool in) {
            const uint32_t cx = in ? (uint32_t)((int)tx + dx) : tx;
            const uint4 v = *reinterpret_cast<const uint4*>(map + ((size_t)cy * n_tx + cx) * kTile + row);
            return in && y_in ? v : make_uint4(0u, 0u, 0u, 0u);
        };
        const bool l_in = tx > 0u, r_in = tx + 1u < n_tx;
        const uint4 pl = rows_at(md.pmap, -1, l_in), pc = rows_at(md.pmap, 0, true), pr = rows_at(md.pmap, 1, r_in);
        const uint4 al = rows_at(rin, -1, l_in), ac = rows_at(rin, 0, true), ar = rows_at(rin, 1, r_in);
        const Row128 pa{{pl.y, pc.x, pc.y, pr.x}}, pb{{pl.w, pc.z, pc.w, pr.z}};
        Row128 a{{al.y, ac.x, ac.y, ar.x}}, b{{al.w, ac.z, ac.w, ar.z}};
        uint32_t plane[5][4] = {};  // of the tile's dwords: row a, then row b
        uint32_t front[4] = {};     // the tile's sites invaded by the last pass
        uint32_t levels = 0;
        struct Core {
            uint32_t v[4];
        };
        auto core = [&]() { return Core{{a.v[1], a.v[2], b.v[1], b.v[2]}}; };
        auto pass = [&]() {
            Row128 above, below;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                above.v[k] = prev_lane(b.v[k]);
                below.v[k] = next_lane(a.v[k]);
            }
            const Row128 na = spread(a, b, above, pa), nb = spread(b, a, below, pb);
            a = na;
            b = nb;
        };
        // passes in groups of eight; the sites new between two of a group's
        // states are those whose pass number has a certain bit
        auto mark = [&](int j, const Core& later, const Core& before) {
#pragma unroll
            for (int k = 0; k < 4; ++k) plane[j][k] |= later.v[k] & ~before.v[k];
        };
#pragma unroll 1
        do {
            const Row128 a0 = a, b0 = b;
            const Core c0 = core();
            Core c2, c4, c6, c7;
            pass();
            const Core c1 = core();
            pass();
            mark(0, c2 = core(), c1);
            pass();
            const Core c3 = core();
            pass();
            mark(0, c4 = core(), c3);
            mark(1, c4, c2);
            pass();
            const Core c5 = core();
            pass();
            mark(0, c6 = core(), c5);
            pass();
            c7 = core();
            pass();
            const Core c8 = core();
            mark(0, c8, c7);
            mark(1, c8, c6);
            mark(2, c8, c4);
            uint32_t ch = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                front[k] = c8.v[k] & ~c7.v[k];
                const uint32_t eight = c8.v[k] & ~c0.v[k];
                if (levels & 8u) plane[3][k] |= eight;
                if (levels & 16u) plane[4][k] |= eight;
                ch |= (a.v[k] ^ a0.v[k]) | (b.v[k] ^ b0.v[k]);
            }
            levels += 8u;
            if (__ballot(ch != 0u) == 0) break;  // the front has died out in these 128 x 128 sites
        } while (levels < kLevels);
        const bool own = lane >= 16u && lane < 48u;  // lanes with the tile's rows
        const uint32_t fresh[4] = {a.v[1] & ~ac.x, a.v[2] & ~ac.y, b.v[1] & ~ac.z, b.v[2] & ~ac.w};
        const uint64_t changed = __ballot(own && (fresh[0] | fresh[1] | fresh[2] | fresh[3]) != 0u);
        // list the tiles that see the front next launch, and this one where
        // it changed (the other map then takes its rows over)
        const uint64_t fl = __ballot(own && (front[0] | front[2]) != 0u), fr = __ballot(own && (front[1] | front[3]) != 0u);
        const uint64_t kTop = 0xffffull << 16, kBot = 0xffffull << 32;
        if (changed && lane < 9u) {
            const int dty = (int)(lane / 3u) - 1, dtx = (int)(lane % 3u) - 1;
            const uint64_t cols = dtx < 0 ? fl : dtx > 0 ? fr : fl | fr;
            const bool want = lane == 4u || (cols & (dty < 0 ? kTop : dty > 0 ? kBot : kTop | kBot)) != 0;
            const int nty = (int)ty + dty, ntx = (int)tx + dtx;
            if (want && nty >= 0 && nty < (int)n_ty && ntx >= 0 && ntx < (int)n_tx) {
                const uint32_t t = (uint32_t)nty * n_tx + (uint32_t)ntx;
                if (atomicExch(&q_out[t], 1u) == 0u) {
                    const uint32_t p = list_part(m, (uint32_t)ntx, (uint32_t)nty);
                    const uint32_t pos = atomicAdd(&w.len[lout * kSubs + p], 1u);
                    list_out[(size_t)p * w.cap + pos] = make_uint2(m, t);
                }
            }
        }
        if (own)
            *reinterpret_cast<uint4*>(rout + (size_t)tile * kTile + row) = make_uint4(a.v[1], a.v[2], b.v[1], b.v[2]);

        // the arrival passes: about two new sites a row
        uint32_t last = 0;
        if (own) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t* const p = md.arr + (size_t)(ty * kTile + row + (uint32_t)(k >> 1)) * L + tx * kTile + 32u * (k & 1);
                for (uint32_t x = fresh[k]; x; x &= x - 1u) {
                    const uint32_t c = (uint32_t)__builtin_ctz(x);
                    uint32_t v = lo + 1u;
#pragma unroll
                    for (int j = 0; j < 5; ++j) v += __builtin_amdgcn_ubfe(plane[j][k], c, 1) << j;
                    p[c] = v;
                    last = max(last, v);
                }
            }
        }
        if (changed) last = wave_max_u32(last);
        if (lane == 0u) {
            TileStat* const st = md.stat + tile;
            atomicAdd(&st->visits, 1u);
            atomicAdd(&st->iterations, levels);
            if (changed) atomicMax(&st->max_arrival, last);
        }
    }
}

// Summaries: the cluster's sites and which lattice edges it touches from the
// invaded map, the largest arrival and the work from the tiles' statistics.
// Blocks of y = m work on medium m, a thread a tile row.
__global__ void __launch_bounds__(kThreads) k_perc_finish(const Medium* __restrict__ media, Result* res) {
    const Medium& md = media[blockIdx.y];
    const uint32_t L = md.L, n_tx = md.n_tx, n_ty = md.n_ty, n_tiles = n_tx * n_ty;
    uint32_t cnt = 0, mx = 0, edges = 0;
    unsigned long long vis = 0, it = 0;
    const uint64_t rows = (uint64_t)n_tiles * kTile, stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t k = (uint64_t)blockIdx.x * kThreads + threadIdx.x; k < rows; k += stride) {
        const uint64_t v = md.reach[0][k];
        const uint32_t t = (uint32_t)(k / kTile), r = (uint32_t)(k % kTile);
        if (r == 0u) {
            const TileStat st = md.stat[t];
            mx = max(mx, st.max_arrival);
            vis += st.visits;
            it += st.iterations;
        }
        if (v == 0) continue;
        const uint32_t ty = t / n_tx, tx = t - ty * n_tx, i = ty * kTile + r;
        cnt += (uint32_t)__builtin_popcountll(v);
        edges |= (i == 0u ? 1u : 0u) | (i == L - 1u ? 2u : 0u) | (tx == 0u && (v & 1u) ? 4u : 0u) |
                 (tx == n_tx - 1u && ((v >> ((L - 1u) % kTile)) & 1u) ? 8u : 0u);
    }
    unsigned long long total = cnt;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        total += __shfl_xor(total, off, 64);
        vis += __shfl_xor(vis, off, 64);
        it += __shfl_xor(it, off, 64);
        mx = max(mx, (uint32_t)__shfl_xor(mx, off, 64));
        edges |= (uint32_t)__shfl_xor(edges, off, 64);
    }
    if ((threadIdx.x & 63u) == 0u) {
        Result* const r = res + blockIdx.y;
        if (total) atomicAdd(&r->invaded, total);
        if (vis) atomicAdd(&r->visits, vis);
        if (it) atomicAdd(&r->iterations, it);
        if (mx) atomicMax(&r->max_arrival, mx);
        if (edges) atomicOr(&r->edges, edges);
    }
}

__global__ void __launch_bounds__(kThreads) k_perc_clear(Result* res, uint32_t count) {
    for (uint32_t m = blockIdx.x * kThreads + threadIdx.x; m < count; m += gridDim.x * kThreads) res[m] = Result{};
}

// Blocks for `work` items of `per` a block, shared with `count` media.
static uint32_t blocks_of(uint64_t work, uint64_t per, uint32_t count) {
    const uint64_t most = count >= 4096u ? 1u : 4096u / count;
    const uint64_t b = (work + per - 1) / per;
    return (uint32_t)(b > most ? most : (b ? b : 1));
}

hipError_t launch_draw(const Medium* media, uint32_t count, uint32_t max_L, const WorkLists& w, Result* res,
                       hipStream_t s) {
    k_perc_clear<<<(count + kThreads - 1) / kThreads, kThreads, 0, s>>>(res, count);
    const uint64_t side = (uint64_t)((max_L + kTile - 1) / kTile) * kTile;
    const uint64_t chunks = side * ((max_L + 255u) / 256u);  // four a block at a time
    for (uint32_t m = 0; m < count; m += 32768u) {            // grid.y is at most 65535
        const uint32_t c = count - m < 32768u ? count - m : 32768u;
        k_perc_draw<<<dim3(blocks_of(chunks, 4, c), c), kThreads, 0, s>>>(media + m, w, res + m);
    }
    return hipGetLastError();
}

hipError_t launch_seed(const Medium* media, uint32_t count, const WorkLists& w, hipStream_t s) {
    k_perc_seed<<<count, kThreads, 0, s>>>(media, w);
    return hipGetLastError();
}

// 32 passes a launch: the most that a border of 32 sites allows.
hipError_t launch_relax(const Medium* one, const Medium* media, const WorkLists& w, uint64_t k, uint32_t grid,
                        hipStream_t s) {
    const uint32_t pin = (uint32_t)(k % 2), lin = (uint32_t)(k % 3), lout = (uint32_t)((k + 1) % 3),
                   lclr = (uint32_t)((k + 2) % 3), lo = (uint32_t)(k * kLevels);
    if (one)
        k_perc_relax<true><<<grid, kRelaxThreads, 0, s>>>(*one, media, w, pin, lin, lout, lclr, lo);
    else
        k_perc_relax<false><<<grid, kRelaxThreads, 0, s>>>(Medium{}, media, w, pin, lin, lout, lclr, lo);
    return hipGetLastError();
}

hipError_t launch_finish(const Medium* media, uint32_t count, uint32_t max_L, Result* res, hipStream_t s) {
    const uint64_t side = (max_L + kTile - 1) / kTile;
    for (uint32_t m = 0; m < count; m += 32768u) {
        const uint32_t c = count - m < 32768u ? count - m : 32768u;
        k_perc_finish<<<dim3(blocks_of(side * side * kTile, 1024, c), c), kThreads, 0, s>>>(media + m, res + m);
    }
    return hipGetLastError();
}

}  // namespace perc
