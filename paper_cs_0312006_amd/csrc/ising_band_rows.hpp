// Band-resident sweeps of one lattice, a wave per row: the lattice is split
// into G bands of whole rows (one workgroup each, all resident at once, as
// in ising_bands.hip), and wave e of a workgroup keeps one row of its band
// for the whole launch: both colours of the row as byte words (four sites a
// word, CW words a lane) in registers, with a copy in LDS for the rows above
// and below.
//
// What bounds such a lattice is latency, not the chip's rate: at 1024^2 a
// half-sweep is one row of two words a lane, and trading edge rows with the
// neighbouring workgroups through memory took two thirds of the 1.6 us it took. So bands
// trade edge rows only every D half-sweeps. A band also updates the rows
// just outside it, as far as they can still be updated from what was traded:
// with the rows at distance 1..D known at the start, half-sweep j = 0 .. D-1
// of the D updates the rows up to distance D - 1 - j. Those rows belong to
// the neighbouring bands, which update them the same way (the draws are keyed
// by site), so both hold the same spins. The extra rows run on waves of
// their own.
//
// A wave has a fixed row, so the parts of its Philox calls that depend only
// on the site (and not on the sweep) are computed once per launch: with
// counter (q, t, c, 0), the products of the first two rounds that involve q
// do not depend on t, nor does one product of the third (see
// SiteDraws). A call is then 32 operations and 8 rounds deep rather than 37
// and 10. The draws of a row's next update do not depend on any spin either:
// for up to four words a lane they are computed before the workgroup barrier
// or the edge wait that precedes the update, off the path that bounds the
// launch.
//
// Rows:
//   kRowsFull    L/8 words fill the 64 CW words of a wave exactly
//   kRowsRagged  L % 8 == 0, fewer words: the word after the last is a copy
//                of word 0 ("ghost"), so that the last word finds its right
//                neighbour where every other word does
//   kRowsShifted any other even L: sites are numbered across rows, so a row
//                starts o = (i H) & 3 bytes into a word (H = L/2 sites of one
//                colour a row) and words stay the sites of one Philox call.
//                Rows above and below are read through a byte shift by the
//                difference of the rows' starts; the bytes just outside the
//                row are ghosts of its other end.
//
// Creutz's demon dynamics (CREUTZ) runs the same way with the demons of a
// row in its wave's registers: they never pass through LDS, and travel with
// the edge rows where bands update rows outside them. It draws nothing, so a
// half-sweep is shorter still against an exchange, and bands of up to ten
// rows trade edges every four half-sweeps. Reversed sweeps take the colours
// in the other order.
//
// Edge rows travel as in ising_bands.hip: 64-bit agent-scope atomics {tag,
// bits}, a lane's CW words as 4 CW bits (both colours in one atomic up to
// four words a lane), double-buffered by the parity of the exchange. The
// exchange number x is published only after the band's waves have read
// exchange x - 1, and they read it only once the neighbour published it,
// which the neighbour did after reading x - 2: the slot it overwrites.
// Rows in HBM are read once at the start, also by the neighbouring bands,
// and written at the end, behind a flag with which each band says that its
// reads are done.
//
// One MI355X, us a sweep over calls of 2048 and more: 64^2 to 512^2 1.39 (at
// 512^2 189 site updates/ns), 1000^2 1.83, 1002^2 2.12, 1024^2 1.79 (586),
// 2048^2 3.02 (1389), 3072^2 5.38, 4096^2 6.88 (2438), with and without a field;
// before and after at each side: row_bands_serve. Up to 1024 the rest is latency
// (an exchange of about 1 us per two sweeps, and per half-sweep two LDS round
// trips, a barrier and one row's 45 to 90 dependent operations); at 4096 the
// four waves of each SIMD keep the vector units busy.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ising_band_edges.hpp"
#include "ising_bands.hpp"
#include "ising_creutz.hpp"
#include "ising_fused_core.hpp"
#include "ising_site_draws.hpp"

namespace ising {

namespace {

constexpr int kRowsFull = 0, kRowsRagged = 1, kRowsShifted = 2;
constexpr uint32_t kMaxRowWaves = 16;
constexpr uint32_t kFlushSweeps = 32;  // sweeps whose wave sums are kept in LDS between flushes

// A row's words as bits (site b of word j at 4 j + b), and back.
template <int CW>
__device__ __forceinline__ uint32_t row_bits(const Row<CW>& r) {
    uint32_t v = 0;
#pragma unroll
    for (int j = 0; j < CW; ++j) v |= ((r.v[j] * 0x01020408u) >> 24) << (4 * j);
    return v;
}
template <int CW>
__device__ __forceinline__ Row<CW> row_of_bits(uint32_t v) {
    Row<CW> r;
#pragma unroll
    for (int j = 0; j < CW; ++j) r.v[j] = (((v >> (4 * j)) & 0xfu) * 0x00204081u) & 0x01010101u;
    return r;
}

// Tagged words a lane publishes of a row: its bits (both colours from D = 2
// up, in one word up to four words a lane) and, Creutz, from D = 2 up the
// demons of both colours.
__host__ __device__ constexpr int bit_entries(int cw, int d) { return d > 1 && cw > 4 ? 2 : 1; }
__host__ __device__ constexpr int entries_per_row(int cw, int d, bool creutz) {
    return bit_entries(cw, d) + (creutz && d > 1 ? 2 * cw : 0);
}

// LDS words of a row-band workgroup of `waves` waves: both planes of every
// wave's row, a word of padding on either side (the shifted rows' reads reach
// one word past a row).
__host__ __device__ constexpr uint32_t row_band_lds_words(uint32_t waves, uint32_t cw) {
    return 2u * waves * 64u * cw + 2u;
}

template <int CW, int MODE, int D, bool CREUTZ>
__global__ __launch_bounds__(1024) void k_band_rows(BandArgs a) {
    constexpr int SE = bit_entries(CW, D), NE = entries_per_row(CW, D, CREUTZ);
    constexpr bool kDemonsTravel = CREUTZ && D > 1;
    constexpr bool kPredraw = CW <= 4 && !CREUTZ;     // draws of the next update kept in registers
    constexpr bool kFixedProduct = CW <= 4 && !CREUTZ;  // both colours' fixed product kept too
    constexpr uint32_t RS = 64u * CW;
    extern __shared__ uint32_t lds[];
    __shared__ LdsTable lt;
    __shared__ uint32_t red[kFlushSweeps][kMaxRowWaves];
    if (!CREUTZ) load_table(lt, a.at);
    const uint32_t first = CREUTZ ? a.rev : 0u;  // the colour of a sweep's first half
    const uint32_t G = gridDim.x, g = blockIdx.x;
    const uint32_t L = a.L, H2 = L / 2u;
    const uint32_t r0 = (uint32_t)((uint64_t)g * L / G);
    const int H = (int)((uint32_t)((uint64_t)(g + 1u) * L / G) - r0);
    const uint32_t lane = threadIdx.x & 63u, nw = blockDim.x >> 6;
    const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t gu = g == 0 ? G - 1u : g - 1u, gd = g + 1u == G ? 0u : g + 1u;
    const uint32_t k0 = a.k0, k1 = a.k1;
    uint32_t* const lat = lds + 1;
    const uint32_t plane_words = nw * RS;

    // this wave's row
    const int lr = (int)e - (D - 1);                               // relative to the band's first row
    const int out = lr < 0 ? -lr : (lr >= H ? lr - H + 1 : 0);    // distance outside the band
    const bool present = out <= D - 1;
    const bool in_band = out == 0;
    const bool top_outer = lr == -(D - 1), bot_outer = lr == H + D - 2;
    int ir = (int)r0 + lr;
    ir = ir < 0 ? ir + (int)L : (ir >= (int)L ? ir - (int)L : ir);
    const uint32_t i = (uint32_t)ir;
    const uint32_t iu = i == 0 ? L - 1u : i - 1u, id = i + 1u == L ? 0u : i + 1u;
    const uint32_t x = lane * (uint32_t)CW;  // the lane's first word of a row

    // word layout of a row: o bytes before its first site, nwd words in use
    auto start_of = [&](uint32_t row) { return MODE == kRowsShifted ? (row * H2) & 3u : 0u; };
    const uint32_t o = start_of(i);
    const uint32_t Hw = MODE == kRowsShifted ? 0u : H2 / 4u;
    const uint32_t q0 = MODE == kRowsShifted ? (i * H2 - o) / 4u : i * Hw;  // the row's first quad
    const int du = MODE == kRowsShifted ? (int)start_of(iu) - (int)o : 0;
    const int dd = MODE == kRowsShifted ? (int)start_of(id) - (int)o : 0;
    // the word (byte) holding the row's last site
    const uint32_t last_pos = MODE == kRowsShifted ? o + H2 - 1u : 4u * Hw - 1u;
    const uint32_t last_col = last_pos / 4u;
    const uint32_t last_lane = last_col / (uint32_t)CW, last_w = last_col % (uint32_t)CW;

    // masks: valid sites (bit 0 of each byte), ghost of the first site (or
    // word) after the last, ghost of the last site before the first
    uint32_t vm[CW], gm[CW], gp = 0;
#pragma unroll
    for (int w = 0; w < CW; ++w) {
        const uint32_t col = x + (uint32_t)w;
        vm[w] = 0x01010101u;
        gm[w] = 0;
        if (MODE == kRowsRagged) {
            if (col >= Hw) vm[w] = 0;
            if (col == Hw) gm[w] = 0x01010101u;
        } else if (MODE == kRowsShifted) {
            uint32_t m = 0, gn = 0;
#pragma unroll
            for (uint32_t b = 0; b < 4u; ++b) {
                const uint32_t pos = 4u * col + b;
                if (pos >= o && pos <= last_pos) m |= 1u << (8u * b);
                if (pos == last_pos + 1u) gn |= 1u << (8u * b);
            }
            vm[w] = m;
            gm[w] = gn;
        }
    }
    if (MODE == kRowsShifted && lane == 0u && o > 0u) gp = 1u << (8u * (o - 1u));

    // A row of a plane from HBM, ghosts included.
    auto load_row = [&](uint32_t row, const uint32_t* plane) {
        Row<CW> r;
        if (MODE == kRowsShifted) {
            const uint8_t* p = reinterpret_cast<const uint8_t*>(plane) + (size_t)row * H2;
            const int so = (int)start_of(row);
#pragma unroll
            for (int w = 0; w < CW; ++w) {
                uint32_t v = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    int m = 4 * ((int)x + w) + b - so;
                    const bool ok = m >= -1 && m <= (int)H2;
                    m = m < 0 ? (int)H2 - 1 : (m == (int)H2 ? 0 : m);
                    if (ok) v |= (uint32_t)p[m] << (8 * b);
                }
                r.v[w] = v;
            }
        } else {
            const uint32_t* p = plane + (size_t)row * Hw;
#pragma unroll
            for (int w = 0; w < CW; ++w) {
                const uint32_t col = x + (uint32_t)w;
                if (MODE == kRowsFull) r.v[w] = p[col];
                else r.v[w] = col < Hw ? p[col] : (col == Hw ? p[0] : 0u);
            }
        }
        return r;
    };
    auto lds_row = [&](uint32_t c, uint32_t row) { return lat + c * plane_words + row * RS + lane; };
    auto put_row = [&](uint32_t c, const Row<CW>& r) {
        uint32_t* p = lds_row(c, e);
#pragma unroll
        for (int w = 0; w < CW; ++w) p[(uint32_t)w * 64u] = r.v[w];
    };
    // Words of a neighbouring row at this row's positions: v[0..CW-1] and
    // the word before (d < 0) or after (d > 0) them, shifted by d bytes.
    auto shift_row = [&](const Row<CW>& v, uint32_t extra, int d) {
        Row<CW> r;
        if (d < 0) {
#pragma unroll
            for (int w = 0; w < CW; ++w)
                r.v[w] = __builtin_amdgcn_alignbyte(v.v[w], w > 0 ? v.v[w > 0 ? w - 1 : 0] : extra, (uint32_t)(4 + d));
        } else {
#pragma unroll
            for (int w = 0; w < CW; ++w)
                r.v[w] = __builtin_amdgcn_alignbyte(w + 1 < CW ? v.v[w + 1 < CW ? w + 1 : 0] : extra, v.v[w], (uint32_t)d);
        }
        return r;
    };
    auto near_lds = [&](uint32_t c, uint32_t row, int d) {
        const uint32_t* p = lds_row(c, row);
        Row<CW> v;
#pragma unroll
        for (int w = 0; w < CW; ++w) v.v[w] = p[(uint32_t)w * 64u];
        if (MODE != kRowsShifted) return v;
        // the extra word: the previous lane's last or the next lane's first
        // (past either end of the row it is not needed, the address stays
        // inside the padded area)
        const uint32_t extra = d < 0 ? p[(int)(CW - 1) * 64 - 1] : p[1];
        return shift_row(v, extra, d);
    };
    auto near_reg = [&](const Row<CW>& v, int d) {
        if (MODE != kRowsShifted) return v;
        const uint32_t extra = d < 0 ? from_left(v.v[CW - 1], 0u) : from_right(v.v[0], 0u);
        return shift_row(v, extra, d);
    };

    Row<CW> own0{}, own1{}, dem0{}, dem1{};
    uint32_t far_u = 0, far_d = 0;  // as bits
    SiteDraws sd[CW];
    uint32_t x0q[CW];
    uint64_t pr0[kFixedProduct ? CW : 1], pr1[kFixedProduct ? CW : 1];
    if (present) {
        own0 = load_row(i, a.p0);
        own1 = load_row(i, a.p1);
        if (CREUTZ) {
            dem0 = load_row(i, a.d0);
            dem1 = load_row(i, a.d1);
        }
    }
    put_row(0u, own0);
    put_row(1u, own1);
    if (threadIdx.x == 0) lds[0] = lds[2u * plane_words + 1u] = 0u;
    // the row beyond the outermost one, in the colour the first half-sweep reads
    if (top_outer) far_u = row_bits<CW>(load_row(iu, first ? a.p0 : a.p1));
    if (bot_outer) far_d = row_bits<CW>(load_row(id, first ? a.p0 : a.p1));
#pragma unroll
    for (int w = 0; w < (CREUTZ ? 0 : CW); ++w) {
        sd[w] = site_draws(q0 + x + (uint32_t)w, k0, k1, x0q[w]);
        if (kFixedProduct) {
            pr0[w] = mul_u64(x0q[w], kPhiloxM0);
            pr1[w] = mul_u64(x0q[w] ^ kPhiloxM1, kPhiloxM0);
        }
    }
    uint4 rr[CW];
    auto draw_word = [&](auto cc, int w, const SweepDraws& s) {
        constexpr int C = decltype(cc)::value;
        const uint64_t p = kFixedProduct ? (C ? pr1[kFixedProduct ? w : 0] : pr0[kFixedProduct ? w : 0])
                                         : mul_u64(C ? x0q[w] ^ kPhiloxM1 : x0q[w], kPhiloxM0);
        return philox_fixed(sd[w], p, s, k0, k1);
    };
    auto draw = [&](auto cc, uint32_t t) {
        const SweepDraws s = sweep_draws(t, k0, k1);
#pragma unroll
        for (int w = 0; w < CW; ++w) rr[w] = draw_word(cc, w, s);
    };
    if (kPredraw && present) draw(Step<0>{}, a.t0);

    // every read of the lattice in HBM has arrived: say so to the neighbours
    uint64_t* const loaded = a.pub + (size_t)2 * G * 2u * D * NE * 64u;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) put_word(loaded + g, a.base + 1u, 1u);

    // the word (kRowsShifted: the byte, in every byte) that ends a row, for
    // the site before its first one
    auto last_of = [&](const Row<CW>& r) {
        if (MODE == kRowsFull) return (uint32_t)__builtin_amdgcn_readlane((int)r.v[CW - 1], 63);
        uint32_t v = 0;
#pragma unroll
        for (int w = 0; w < CW; ++w)
            if (last_w == (uint32_t)w) v = (uint32_t)__builtin_amdgcn_readlane((int)r.v[w], (int)last_lane);
        if (MODE == kRowsShifted) v = ((v >> (8u * (last_pos & 3u))) & 1u) * 0x01010101u;
        return v;
    };

    const bool top_pub = in_band && lr < D, bot_pub = in_band && lr >= H - D;
    auto slot = [&](uint32_t par, uint32_t band, uint32_t edge, uint32_t dist) {
        return a.pub + ((((size_t)par * G + band) * 2u + edge) * D + dist) * NE * 64u + lane;
    };
    auto publish = [&](uint32_t par, uint32_t edge, uint32_t dist, uint32_t tag, uint32_t c_last) {
        uint64_t* p = slot(par, g, edge, dist);
        if (D == 1) {
            put_word(p, tag, c_last ? row_bits<CW>(own1) : row_bits<CW>(own0));
        } else if (SE == 1) {
            put_word(p, tag, row_bits<CW>(own0) | (row_bits<CW>(own1) << 16));
        } else {
            put_word(p, tag, row_bits<CW>(own0));
            put_word(p + 64, tag, row_bits<CW>(own1));
        }
        if (kDemonsTravel && dist < D - 1u) {
#pragma unroll
            for (int w = 0; w < CW; ++w) {
                put_word(p + 64 * (SE + w), tag, dem0.v[w]);
                put_word(p + 64 * (SE + CW + w), tag, dem1.v[w]);
            }
        }
    };

    // One half-sweep of this wave's row: colour C, the sweep's first or second
    // half, step J of the D between two exchanges, sweep t, sweep number s of
    // the launch.
    auto update = [&](auto cc, auto half, auto jj, uint32_t t, uint32_t s) {
        constexpr int C = decltype(cc)::value, J = decltype(jj)::value;
        constexpr bool kSecond = decltype(half)::value == 1;
        Row<CW>& own = C ? own1 : own0;
        Row<CW>& dem = C ? dem1 : dem0;
        const Row<CW>& same = C ? own0 : own1;
        Row<CW> up, dn;
        if (J == 0 && top_outer) up = near_reg(row_of_bits<CW>(far_u), du);
        else up = near_lds(1u - C, e - 1u, du);
        if (J == 0 && bot_outer) dn = near_reg(row_of_bits<CW>(far_d), dd);
        else dn = near_lds(1u - C, e + 1u, dd);
        const SweepDraws sw = CREUTZ ? SweepDraws{0u, 0u} : sweep_draws(t, k0, k1);
        Row<CW> S;
        if ((i + (uint32_t)C) & 1u) {
            const uint32_t edge = MODE == kRowsFull ? (uint32_t)__builtin_amdgcn_readlane((int)same.v[0], 0) : 0u;
            const uint32_t nb = from_right(same.v[0], edge);
#pragma unroll
            for (int w = 0; w < CW; ++w)
                S.v[w] = __builtin_amdgcn_alignbyte(w + 1 < CW ? same.v[w + 1 < CW ? w + 1 : 0] : nb, same.v[w], 1);
        } else {
            const uint32_t nb = from_left(same.v[CW - 1], last_of(same));
#pragma unroll
            for (int w = 0; w < CW; ++w)
                S.v[w] = __builtin_amdgcn_alignbyte(same.v[w], w > 0 ? same.v[w > 0 ? w - 1 : 0] : nb, 3);
        }
        uint32_t sad = 0, ups = 0;
#pragma unroll
        for (int w = 0; w < CW; ++w) {
            const uint32_t n = up.v[w] + dn.v[w] + S.v[w] + same.v[w];
            uint32_t nv;
            if (CREUTZ) {
                creutz_word(own.v[w], n, dem.v[w], nv, dem.v[w]);
            } else {
                const AcceptEntries ent = accept_entries(lt, (own.v[w] << 3) + n);
                if (kPredraw) {
                    nv = accept_from(ent, rr[w]);
                } else {
                    __builtin_amdgcn_sched_barrier(0);  // the table reads stay ahead of the Philox call
                    nv = accept_from(ent, draw_word(cc, w, sw));
                }
            }
            if (MODE != kRowsFull) nv &= vm[w];
            if (kSecond) {
                sad = sad_misaligned(nv, MODE == kRowsFull ? n : n & ((vm[w] << 3) - vm[w]), sad);
                ups += nv + (MODE == kRowsFull ? same.v[w] : same.v[w] & vm[w]);  // bytewise, at most 16
            }
            own.v[w] = nv;
        }
        if (MODE == kRowsRagged) {
            const uint32_t head = (uint32_t)__builtin_amdgcn_readlane((int)own.v[0], 0);
#pragma unroll
            for (int w = 0; w < CW; ++w) own.v[w] |= head & gm[w];
        } else if (MODE == kRowsShifted) {
            const uint32_t head = (((uint32_t)__builtin_amdgcn_readlane((int)own.v[0], 0) >> (8u * o)) & 1u) * 0x01010101u;
            const uint32_t last = last_of(own);
#pragma unroll
            for (int w = 0; w < CW; ++w) own.v[w] |= head & gm[w];
            own.v[0] |= last & gp;
        }
        put_row(C, own);
        if (kSecond && in_band) {
            // a row's sums fit 16 bits each: sad <= 4 per site, ups <= 1
            const uint32_t both = wave_sum_lane63(sad | (__builtin_amdgcn_sad_u8(ups, 0u, 0u) << 16));
            if (lane == 63u) red[s % kFlushSweeps][e] = both;
        }
    };
    // flush `count` sweeps ending before sweep `end` of the launch
    auto flush = [&](uint32_t end, uint32_t count) {
        if (threadIdx.x < count) {
            const uint32_t s = end - count + threadIdx.x;
            int64_t sm = 0, su = 0;
            for (int w = 0; w < H; ++w) {
                const uint32_t v = red[s % kFlushSweeps][w + D - 1];
                sm += v & 0xffffu;
                su += v >> 16;
            }
            const int64_t HL = (int64_t)H * L;  // the band's sites: 2 H L bonds, each counted once
            int64_t* p = a.part + 2u * ((size_t)s * G + g);
            p[0] = 2 * HL - 2 * sm;
            p[1] = 2 * su - HL;
        }
    };

    const uint32_t halves = 2u * a.n;
    uint32_t flushed = 0;
    // step J of a block of D half-sweeps starting at half-sweep tau0, a
    // sweep's first (half = 0) or second half
    auto step = [&](auto half, auto jj, uint32_t tau0) {
        constexpr int C = decltype(half)::value, J = decltype(jj)::value;  // C: the colour, unless reversed
        const uint32_t tau = tau0 + J, s = tau >> 1;
        if (tau >= halves) return;
        const bool more = tau0 + D < halves;  // another block follows
        const uint32_t par = ((tau0 / D) + 1u) & 1u, tag = a.base + tau0 + D;
        if (present && out <= D - 1 - J) {
            if (CREUTZ && first) update(Step<1 - C>{}, half, jj, a.t0 + s, s);
            else update(Step<C>{}, half, jj, a.t0 + s, s);
            if (J == D - 1 && more) {
                if (top_pub) publish(par, 0u, (uint32_t)lr, tag, C ^ first);
                if (bot_pub) publish(par, 1u, (uint32_t)(H - 1 - lr), tag, C ^ first);
            }
            // the next update's draws (in this block or the next one) need no
            // spins: they pass before the barrier and the edge wait
            if (kPredraw) {
                if (J + 1 < D && out <= D - 2 - J) draw(Step<1 - C>{}, a.t0 + ((tau + 1u) >> 1));
                else draw(Step<D == 1 ? 1 - C : 0>{}, a.t0 + ((tau0 + D) >> 1));
            }
        }
        if (J < D - 1 || !more) {
            __syncthreads();
        } else if (D == 1) {
            __syncthreads();  // only the edge rows wait for the neighbours
            if (top_outer || bot_outer) {
                const uint64_t *const u = slot(par, gu, 1u, 0u), *const d = slot(par, gd, 0u, 0u);
                const uint64_t* const ps[2] = {top_outer ? u : d, bot_outer ? d : u};
                uint32_t v[2];
                take_words<2>(ps, tag, a.err, v);
                far_u = v[0];
                far_d = v[1];
            }
        } else {
            if (present && !in_band) {
                // this wave's own row, outside the band, and, for the outermost
                // ones, the row beyond it in the colour a sweep's first half reads
                const uint64_t* const p = lr < 0 ? slot(par, gu, 1u, (uint32_t)(-lr - 1)) : slot(par, gd, 0u, (uint32_t)(lr - H));
                const uint64_t* const far = (lr < 0 ? slot(par, gu, 1u, D - 1) : slot(par, gd, 0u, D - 1)) +
                                            (SE == 2 && !first ? 64 : 0);
                constexpr int N = NE + 1;
                const uint64_t* ps[N];
                uint32_t v[N];
#pragma unroll
                for (int k = 0; k < NE; ++k) ps[k] = p + 64 * k;
                ps[NE] = top_outer || bot_outer ? far : p;
                take_words<N>(ps, tag, a.err, v);
                if (SE == 1) {
                    own0 = row_of_bits<CW>(v[0] & 0xffffu);
                    own1 = row_of_bits<CW>(v[0] >> 16);
                } else {
                    own0 = row_of_bits<CW>(v[0]);
                    own1 = row_of_bits<CW>(v[SE - 1]);
                }
                if (kDemonsTravel) {
#pragma unroll
                    for (int w = 0; w < CW; ++w) {
                        dem0.v[w] = v[kDemonsTravel ? SE + w : 0];
                        dem1.v[w] = v[kDemonsTravel ? SE + CW + w : 0];
                    }
                }
                far_u = far_d = SE == 2 ? v[NE] : (first ? v[NE] & 0xffffu : v[NE] >> 16);
            }
            __syncthreads();  // the rows outside the band were read by the last half-sweeps
            if (present && !in_band) {
                put_row(0u, own0);
                put_row(1u, own1);
            }
            __syncthreads();
        }
        if (C && (J == D - 1 || D == 1)) {
            const uint32_t done = s + 1u;
            if (done - flushed == kFlushSweeps) {
                flush(done, kFlushSweeps);
                flushed = done;
            }
        }
    };

    if (D == 1) {
        for (uint32_t tau = 0; tau < halves; tau += 2u) {
            step(Step<0>{}, Step<0>{}, tau);
            step(Step<1>{}, Step<0>{}, tau + 1u);
        }
    } else {
        for (uint32_t tau = 0; tau < halves; tau += D) {
            step(Step<0>{}, Step<0>{}, tau);
            step(Step<1>{}, Step<D == 1 ? 0 : 1>{}, tau);
            if (D == 4) {
                step(Step<0>{}, Step<D == 4 ? 2 : 0>{}, tau);
                step(Step<1>{}, Step<D == 4 ? 3 : 0>{}, tau);
            }
        }
    }
    if (a.n > flushed) flush(a.n, a.n - flushed);

    // the neighbours have read this band's rows: write them back
    if (lane == 0u && e == 0u) {
        (void)take_word(loaded + gu, a.base + 1u, a.err);
        (void)take_word(loaded + gd, a.base + 1u, a.err);
    }
    __syncthreads();
    auto store_row = [&](uint32_t* plane, const Row<CW>& r, uint32_t keep) {
        if (MODE == kRowsShifted) {
            uint8_t* p = reinterpret_cast<uint8_t*>(plane) + (size_t)i * H2;
#pragma unroll
            for (int w = 0; w < CW; ++w)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (vm[w] & (1u << (8 * b))) p[4 * ((int)x + w) + b - (int)o] = (uint8_t)((r.v[w] >> (8 * b)) & keep);
        } else {
            uint32_t* p = plane + (size_t)i * Hw;
#pragma unroll
            for (int w = 0; w < CW; ++w)
                if (MODE == kRowsFull || vm[w]) p[x + (uint32_t)w] = r.v[w];
        }
    };
    if (in_band) {
        store_row(a.p0, own0, 1u);
        store_row(a.p1, own1, 1u);
        if (CREUTZ) {
            store_row(a.d0, dem0, 0xffu);
            store_row(a.d1, dem1, 0xffu);
        }
    }
}

}  // namespace
}  // namespace ising
