// C ABI of the percolation engine (include/percolation.h): contexts, device
// buffers, and the host loop that relaunches the tile relaxation until no
// tile of any medium of the run is listed.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "ising_hostcopy.hpp"
#include "perc_launch.hpp"
#include "percolation.h"

using namespace perc;

namespace {

// What a run needs beside its media: the media table and the results (device
// and pinned host copies), the work lists, and the pinned counts polled
// between launch groups. Owned by the context that runs (a batch: its first
// context), grown to the largest run it has made, freed with it.
struct Workspace {
    size_t media = 0;       // media it has room for
    uint64_t entries = 0;   // work list entries a part has room for
    Medium* d_table = nullptr;
    Medium* h_table = nullptr;
    Result* d_res = nullptr;
    Result* h_res = nullptr;
    uint32_t* h_len = nullptr;  // kSubs counts of each of two launch groups
    hipEvent_t polled[2] = {nullptr, nullptr};
    WorkLists w{};
};

}  // namespace

struct perc_ctx {
    perc_params p{};
    uint64_t N = 0;
    uint32_t n_tx = 0, n_ty = 0, n_tiles = 0;
    int device = 0;
    hipStream_t stream = nullptr;
    bool owns_stream = false;
    uint8_t* pore = nullptr;
    uint32_t* arr = nullptr;
    uint64_t* maps = nullptr;  // pores, and the invaded sites of even and odd launches: 64 words a tile each
    TileStat* stat = nullptr;    // per tile, behind the maps
    uint32_t* queued = nullptr;  // two flags a tile, behind the statistics
    Workspace ws{};
    Result res{};  // of the last run
    uint32_t launches = 0;
    bool ran = false;
    bool poisoned = false;
};

namespace {

// Relaxation launches between polls: a quarter of those made so far, from
// kMinGroup to kMaxGroup. The next group is queued before a group's poll is
// waited for, so the GPU never waits for the host; at most two groups of
// empty launches (2-3 us each) run after the work list is empty.
constexpr uint32_t kMinGroup = 4;
constexpr uint32_t kMaxGroup = 32;
constexpr uint64_t kMaxLaunches = 1ull << 26;  // far beyond any medium: a guard, not a limit

bool valid(const perc_params* p) {
    if (!p || p->L < 1 || p->L > 65536u) return false;
    if (!(p->porosity >= 0.0 && p->porosity <= 1.0)) return false;
    if (p->source > PERC_SOURCE_POINT) return false;
    if (p->source == PERC_SOURCE_POINT && (p->i0 >= p->L || p->j0 >= p->L)) return false;
    return true;
}

int fail(perc_ctx* c) {
    c->poisoned = true;
    (void)hipGetLastError();
    return ISING_EDEVICE;
}

#define PERC_TRY(c, expr)                         \
    do {                                          \
        if ((expr) != hipSuccess) return fail(c); \
    } while (0)

int enter(perc_ctx* c) {
    if (!c) return ISING_EINVAL;
    if (c->poisoned) return ISING_ESTATE;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c);
    return ISING_OK;
}

template <typename T>
bool dev_alloc(T** p, size_t bytes) {
    if (hipMalloc((void**)p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return false;
    }
    return true;
}

uint64_t fnv1a64(const uint8_t* p, size_t n) {
    uint64_t h = 0xcbf29ce484222325ull;
    for (size_t k = 0; k < n; ++k) {
        h ^= p[k];
        h *= 0x100000001b3ull;
    }
    return h;
}

void release(Workspace& ws) {
    (void)hipFree(ws.d_table);
    (void)hipFree(ws.d_res);
    (void)hipFree(ws.w.list[0]);
    (void)hipFree(ws.w.list[1]);
    (void)hipFree(ws.w.len);
    if (ws.h_table) (void)hipHostFree(ws.h_table);
    if (ws.h_res) (void)hipHostFree(ws.h_res);
    if (ws.h_len) (void)hipHostFree(ws.h_len);
    for (hipEvent_t ev : ws.polled)
        if (ev) (void)hipEventDestroy(ev);
    ws = Workspace{};
}

template <typename T>
bool host_alloc(T** p, size_t bytes) {
    if (hipHostMalloc((void**)p, bytes, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return false;
    }
    return true;
}

// Room for `media` media whose work lists take `entries` entries a part.
// Nothing is queued on it when a run starts (runs synchronise).
int reserve(Workspace& ws, size_t media, uint64_t entries) {
    if (media <= ws.media && entries <= ws.entries) return ISING_OK;
    const size_t m = std::max(media, ws.media);
    const uint64_t n = std::max(entries, ws.entries);
    release(ws);
    bool ok = dev_alloc(&ws.d_table, m * sizeof(Medium)) && dev_alloc(&ws.d_res, m * sizeof(Result)) &&
              dev_alloc(&ws.w.list[0], kSubs * n * sizeof(uint2)) &&
              dev_alloc(&ws.w.list[1], kSubs * n * sizeof(uint2)) &&
              dev_alloc(&ws.w.len, 3 * kSubs * sizeof(uint32_t)) && host_alloc(&ws.h_table, m * sizeof(Medium)) &&
              host_alloc(&ws.h_res, m * sizeof(Result)) && host_alloc(&ws.h_len, 2 * kSubs * sizeof(uint32_t));
    for (hipEvent_t& ev : ws.polled)
        if (ok && hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            ev = nullptr;
            ok = false;
        }
    if (!ok) {
        release(ws);
        return ISING_ENOMEM;
    }
    ws.media = m;
    ws.entries = n;
    ws.w.cap = (uint32_t)n;
    return ISING_OK;
}

// One-wave workgroups of a relaxation launch: one per tile, at most 16 per
// compute unit, a multiple of the list's parts.
uint32_t relax_grid(uint64_t tiles, int device) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0) {
        (void)hipGetLastError();
        cus = 256;
    }
    const uint64_t g = std::min<uint64_t>(tiles, (uint64_t)cus * 16u);
    return (uint32_t)((g + kSubs - 1) / kSubs * kSubs);
}

Medium describe(const perc_ctx* c) {
    const size_t words = (size_t)c->n_tiles * kTile;
    Medium m{};
    m.pore = c->pore;
    m.arr = c->arr;
    m.pmap = c->maps;
    m.reach[0] = c->maps + words;
    m.reach[1] = c->maps + 2 * words;
    m.queued[0] = c->queued;
    m.queued[1] = c->queued + c->n_tiles;
    m.stat = c->stat;
    m.pthr = (uint64_t)std::floor(c->p.porosity * 4294967296.0);
    m.L = c->p.L;
    m.n_tx = c->n_tx;
    m.n_ty = c->n_ty;
    m.k0 = (uint32_t)c->p.seed;
    m.k1 = (uint32_t)(c->p.seed >> 32);
    m.source = c->p.source;
    m.i0 = c->p.i0;
    m.j0 = c->p.j0;
    return m;
}

// Draw and invade the media ctxs[0..count) on stream s with the workspace
// and device of ctxs[0]. Synchronises s. Errors poison ctxs[0].
int run_media(perc_ctx* const* ctxs, size_t count, hipStream_t s) {
    perc_ctx* c0 = ctxs[0];
    uint64_t entries = 0, tiles = 0;
    uint32_t max_L = 0;
    for (size_t m = 0; m < count; ++m) {
        entries += part_entries(ctxs[m]->p.L);
        tiles += ctxs[m]->n_tiles;
        max_L = std::max(max_L, ctxs[m]->p.L);
    }
    if (entries > 0xffffffffu / kSubs) return ISING_ERANGE;  // list positions are 32 bits
    Workspace& ws = c0->ws;
    const int rc = reserve(ws, count, entries);
    if (rc != ISING_OK) return rc;
    for (size_t m = 0; m < count; ++m) {
        ctxs[m]->ran = false;
        ws.h_table[m] = describe(ctxs[m]);
    }
    PERC_TRY(c0, hipMemcpyAsync(ws.d_table, ws.h_table, count * sizeof(Medium), hipMemcpyHostToDevice, s));
    PERC_TRY(c0, launch_draw(ws.d_table, (uint32_t)count, max_L, ws.w, ws.d_res, s));
    PERC_TRY(c0, launch_seed(ws.d_table, (uint32_t)count, ws.w, s));
    const uint32_t grid = relax_grid(tiles, c0->device);
    uint64_t k = 0;
    auto queue_group = [&](uint32_t slot) -> hipError_t {
        const uint32_t group = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(k / 4u, kMinGroup), kMaxGroup);
        for (uint32_t g = 0; g < group; ++g, ++k) {
            const hipError_t r = launch_relax(count == 1 ? ws.h_table : nullptr, ws.d_table, ws.w, k, grid, s);
            if (r != hipSuccess) return r;
        }
        // the entries queued for launch k
        const hipError_t r = hipMemcpyAsync(ws.h_len + slot * kSubs, ws.w.len + (k % 3) * kSubs,
                                            kSubs * sizeof(uint32_t), hipMemcpyDeviceToHost, s);
        return r != hipSuccess ? r : hipEventRecord(ws.polled[slot], s);
    };
    PERC_TRY(c0, queue_group(0));
    for (uint32_t slot = 0;; slot ^= 1u) {
        if (k >= kMaxLaunches) return ISING_ERANGE;
        PERC_TRY(c0, queue_group(slot ^ 1u));
        PERC_TRY(c0, hipEventSynchronize(ws.polled[slot]));
        bool empty = true;
        for (uint32_t p = 0; p < kSubs; ++p) empty = empty && ws.h_len[slot * kSubs + p] == 0;
        if (empty) break;
    }
    PERC_TRY(c0, launch_finish(ws.d_table, (uint32_t)count, max_L, ws.d_res, s));
    PERC_TRY(c0, hipMemcpyAsync(ws.h_res, ws.d_res, count * sizeof(Result), hipMemcpyDeviceToHost, s));
    PERC_TRY(c0, hipStreamSynchronize(s));
    for (size_t m = 0; m < count; ++m) {
        ctxs[m]->res = ws.h_res[m];
        ctxs[m]->launches = (uint32_t)std::min<uint64_t>(k, 0xffffffffu);
        ctxs[m]->ran = true;
    }
    return ISING_OK;
}

}  // namespace

extern "C" {

int perc_create(const perc_params* params, void* stream, perc_ctx** out) {
    if (!out) return ISING_EINVAL;
    *out = nullptr;
    if (!valid(params)) return ISING_EINVAL;
    perc_ctx* c = new (std::nothrow) perc_ctx();
    if (!c) return ISING_ENOMEM;
    c->p = *params;
    const uint32_t L = params->L;
    c->N = (uint64_t)L * L;
    c->n_tx = (L + kTile - 1) / kTile;
    c->n_ty = c->n_tx;
    c->n_tiles = c->n_tx * c->n_ty;
    ising::hostcopy_retain();
    if (hipGetDevice(&c->device) != hipSuccess) {
        ising::hostcopy_release();
        delete c;
        return ISING_EDEVICE;
    }
    if (stream) {
        c->stream = (hipStream_t)stream;
    } else {
        if (hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking) != hipSuccess) {
            ising::hostcopy_release();
            delete c;
            return ISING_EDEVICE;
        }
        c->owns_stream = true;
    }
    const bool ok = dev_alloc(&c->pore, c->N) && dev_alloc(&c->arr, c->N * sizeof(uint32_t)) &&
                    dev_alloc(&c->maps, (size_t)c->n_tiles * (3 * kTile * sizeof(uint64_t) + sizeof(TileStat) +
                                                              2 * sizeof(uint32_t)));
    if (!ok) {
        perc_destroy(c);
        return ISING_ENOMEM;
    }
    c->stat = reinterpret_cast<TileStat*>(c->maps + (size_t)c->n_tiles * 3 * kTile);
    c->queued = reinterpret_cast<uint32_t*>(c->stat + c->n_tiles);
    *out = c;
    return ISING_OK;
}

int perc_run(perc_ctx* c) {
    int rc = enter(c);
    if (rc != ISING_OK) return rc;
    return run_media(&c, 1, c->stream);
}

int perc_run_batch(perc_ctx* const* ctxs, size_t count) {
    if (!ctxs) return ISING_EINVAL;
    if (count == 0) return ISING_OK;
    uint64_t tiles = 0;
    for (size_t m = 0; m < count; ++m) {
        if (!ctxs[m]) return ISING_EINVAL;
        if (ctxs[m]->poisoned) return ISING_ESTATE;
        if (ctxs[m]->device != ctxs[0]->device) return ISING_EINVAL;
        for (size_t j = 0; j < m; ++j)
            if (ctxs[j] == ctxs[m]) return ISING_EINVAL;  // one context may appear once
        tiles += ctxs[m]->n_tiles;
    }
    if (tiles > 0xffffffffu) return ISING_ERANGE;
    perc_ctx* c0 = ctxs[0];
    int rc = enter(c0);
    if (rc != ISING_OK) return rc;
    hipStream_t s = c0->stream;
    // the run starts after each medium's earlier work on its own stream
    for (size_t m = 1; m < count; ++m)
        if (ctxs[m]->stream != s) PERC_TRY(c0, hipStreamSynchronize(ctxs[m]->stream));
    return run_media(ctxs, count, s);
}

int perc_set_params(perc_ctx* c, const perc_params* params) {
    if (!c) return ISING_EINVAL;
    if (c->poisoned) return ISING_ESTATE;
    if (!valid(params) || params->L != c->p.L) return ISING_EINVAL;
    c->p = *params;
    c->ran = false;
    return ISING_OK;
}

int perc_copy_medium(perc_ctx* c, uint8_t* host, size_t n) {
    int rc = enter(c);
    if (rc != ISING_OK) return rc;
    if (!host || n < c->N) return ISING_EINVAL;
    if (!c->ran) return ISING_ESTATE;
    PERC_TRY(c, ising::copy_to_host(host, c->pore, c->N, c->stream));
    return ISING_OK;
}

int perc_copy_arrival(perc_ctx* c, int32_t* host, size_t n) {
    int rc = enter(c);
    if (rc != ISING_OK) return rc;
    if (!host || n < c->N) return ISING_EINVAL;
    if (!c->ran) return ISING_ESTATE;
    PERC_TRY(c, ising::copy_to_host(host, c->arr, c->N * sizeof(int32_t), c->stream));
    return ISING_OK;
}

int perc_result_get(perc_ctx* c, perc_result* out, uint32_t want_hash) {
    int rc = enter(c);
    if (rc != ISING_OK) return rc;
    if (!out) return ISING_EINVAL;
    if (!c->ran) return ISING_ESTATE;
    const Result& st = c->res;
    perc_result r{};
    r.pores = st.pores;
    r.invaded = st.invaded;
    r.passes = (int32_t)st.max_arrival;
    r.spans = ((st.edges & 3u) == 3u ? 1u : 0u) | ((st.edges & 12u) == 12u ? 2u : 0u);
    r.launches = c->launches;
    r.tile_visits = st.visits;
    r.tile_iterations = st.iterations;
    if (want_hash) {
        std::vector<int32_t> a;
        try {
            a.resize(c->N);
        } catch (...) {
            return ISING_ENOMEM;
        }
        rc = perc_copy_arrival(c, a.data(), a.size());
        if (rc != ISING_OK) return rc;
        r.arrival_hash = fnv1a64(reinterpret_cast<const uint8_t*>(a.data()), a.size() * sizeof(int32_t));
    }
    *out = r;
    return ISING_OK;
}

int perc_destroy(perc_ctx* c) {
    if (!c) return ISING_OK;
    (void)hipSetDevice(c->device);
    if (c->stream) (void)hipStreamSynchronize(c->stream);
    (void)hipFree(c->pore);
    (void)hipFree(c->arr);
    (void)hipFree(c->maps);
    release(c->ws);
    if (c->owns_stream && c->stream) (void)hipStreamDestroy(c->stream);
    (void)hipGetLastError();
    ising::hostcopy_release();
    delete c;
    return ISING_OK;
}

}  // extern "C"
