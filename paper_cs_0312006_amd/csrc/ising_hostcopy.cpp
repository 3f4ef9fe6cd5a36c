// Device to pageable host memory through pinned chunks and several threads.
//
// The runtime copies to pageable memory through pinned chunks of its own, one
// at a time, with one thread that moves each chunk into the caller's pages
// (often touched for the first time): 10 GB/s, of the 57 the link carries.
// Here the link fills a ring of pinned chunks while several threads empty
// them.
//
// The ring: chunk c uses slot c % kSlots, is enqueued on the caller's stream
// with an event behind it, and is moved by whichever thread takes number c.
// That thread then enqueues chunk c + kSlots into the slot it has emptied.
// slot_chunk[slot] names the chunk enqueued there last, so a thread that is
// ahead waits for its slot.
//
// Whole calls: 1 GiB (32768^2 spins) 104 -> 27.7 ms, 64 MiB (8192^2) 6.5 ->
// 2.0, 16 MiB (4096^2) 1.0 -> 0.55.
#include "ising_hostcopy.hpp"

#include <sched.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

namespace ising {

namespace {

constexpr size_t kChunk = (size_t)2 << 20;
constexpr uint32_t kSlots = 8;
constexpr size_t kStageBytes = kChunk * kSlots;
constexpr uint32_t kMaxStages = 2;
constexpr uint32_t kMaxThreads = 8;
// Below this the runtime's own path is kept: at 4 MiB the ring still wins
// (0.20 against 0.28 ms) but a process's first copy pays 1 ms for the stage;
// at 16 MiB its first copy takes the same (2.1 against 2.0 ms) and the later
// ones half. At 1 MiB the ring loses (0.17 against 0.09 ms).
constexpr size_t kMinBytes = (size_t)16 << 20;

struct Stage {
    char* mem = nullptr;
    hipEvent_t landed[kSlots] = {};
    int device = -1;  // the events' device
};

std::mutex g_mu;
std::vector<Stage*> g_idle;
uint32_t g_stages = 0, g_users = 0;

void destroy(Stage* st) {
    for (hipEvent_t e : st->landed)
        if (e) (void)hipEventDestroy(e);
    if (st->mem) (void)hipHostFree(st->mem);
    (void)hipGetLastError();
    delete st;
}

// A stage for `device`, or nullptr (all in use, or no pinned memory).
Stage* acquire(int device) {
    Stage* old = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        for (size_t k = 0; k < g_idle.size(); ++k)
            if (g_idle[k]->device == device) {
                Stage* st = g_idle[k];
                g_idle.erase(g_idle.begin() + (ptrdiff_t)k);
                return st;
            }
        if (g_stages >= kMaxStages) {
            if (g_idle.empty()) return nullptr;
            old = g_idle.back();  // another device's: replaced
            g_idle.pop_back();
        } else {
            ++g_stages;
        }
    }
    if (old) destroy(old);
    Stage* st = new (std::nothrow) Stage();
    bool ok = st != nullptr;
    if (ok) {
        st->device = device;
        ok = hipHostMalloc((void**)&st->mem, kStageBytes, hipHostMallocDefault) == hipSuccess;
        if (!ok) st->mem = nullptr;
        for (hipEvent_t& e : st->landed)
            if (ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                e = nullptr;
                ok = false;
            }
    }
    if (!ok) {
        (void)hipGetLastError();
        if (st) destroy(st);
        std::lock_guard<std::mutex> lock(g_mu);
        --g_stages;
        return nullptr;
    }
    return st;
}

void give_back(Stage* st) {
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (g_users > 0 && g_idle.size() < g_idle.capacity()) {  // room reserved by hostcopy_retain
            g_idle.push_back(st);
            return;
        }
        --g_stages;
    }
    destroy(st);
}

uint32_t host_threads() {
    static const uint32_t n = [] {
        cpu_set_t set;
        const int c = sched_getaffinity(0, sizeof(set), &set) == 0 ? CPU_COUNT(&set) : 1;
        return (uint32_t)std::max(1, std::min<int>(c, (int)kMaxThreads));
    }();
    return n;
}

// Whether the link can write to p itself (pinned, managed or device memory).
bool known_to_hip(const void* p) {
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type != hipMemoryTypeUnregistered;
    (void)hipGetLastError();
    return false;
}

struct Ring {
    Stage* st;
    char* dst;
    const char* src;
    size_t bytes;
    hipStream_t s;
    int device;
    uint64_t chunks;
    std::atomic<uint64_t> next{0};
    std::atomic<uint64_t> slot_chunk[kSlots];
    std::atomic<int> error{(int)hipSuccess};

    size_t size(uint64_t c) const { return std::min(kChunk, bytes - (size_t)c * kChunk); }
    void fail(hipError_t e) {
        int none = (int)hipSuccess;
        error.compare_exchange_strong(none, (int)e);
    }
    bool enqueue(uint64_t c) {
        const uint32_t k = (uint32_t)(c % kSlots);
        hipError_t e = hipMemcpyAsync(st->mem + k * kChunk, src + c * kChunk, size(c), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipEventRecord(st->landed[k], s);
        if (e != hipSuccess) fail(e);
        slot_chunk[k].store(c, std::memory_order_release);
        return e == hipSuccess;
    }
    // `helper`: not the calling thread, whose device is set and which moves
    // whatever chunks the helpers do not take.
    void work(bool helper) {
        if (helper && hipSetDevice(device) != hipSuccess) return;
        for (;;) {
            const uint64_t c = next.fetch_add(1, std::memory_order_relaxed);
            if (c >= chunks || error.load(std::memory_order_relaxed) != (int)hipSuccess) return;
            const uint32_t k = (uint32_t)(c % kSlots);
            while (slot_chunk[k].load(std::memory_order_acquire) != c) {
                if (error.load(std::memory_order_relaxed) != (int)hipSuccess) return;
                sched_yield();
            }
            const hipError_t e = hipEventSynchronize(st->landed[k]);
            if (e != hipSuccess) return fail(e);
            memcpy(dst + c * kChunk, st->mem + k * kChunk, size(c));
            if (c + kSlots < chunks) enqueue(c + kSlots);
        }
    }
};

}  // namespace

void hostcopy_retain() {
    std::lock_guard<std::mutex> lock(g_mu);
    try {
        g_idle.reserve(kMaxStages);
    } catch (...) {  // give_back then frees instead of keeping
    }
    ++g_users;
}

void hostcopy_release() {
    std::vector<Stage*> idle;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (--g_users > 0) return;
        idle.swap(g_idle);
        g_stages -= (uint32_t)idle.size();
    }
    for (Stage* st : idle) destroy(st);
}

hipError_t copy_to_host(void* dst, const void* src, size_t bytes, hipStream_t s) {
    int device = 0;
    Stage* st = nullptr;
    // straight into memory that the link can write to: 4096^2 0.35 ms against
    // 0.55 through the ring, 16384^2 5.3 against 6.7, 32768^2 20.9 against 26.6
    if (bytes >= kMinBytes && !known_to_hip(dst) && hipGetDevice(&device) == hipSuccess) st = acquire(device);
    if (!st) {
        const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
        return e != hipSuccess ? e : hipStreamSynchronize(s);
    }
    Ring r;
    r.st = st;
    r.dst = static_cast<char*>(dst);
    r.src = static_cast<const char*>(src);
    r.bytes = bytes;
    r.s = s;
    r.device = device;
    r.chunks = (bytes + kChunk - 1) / kChunk;
    for (auto& c : r.slot_chunk) c.store(~(uint64_t)0, std::memory_order_relaxed);
    bool ok = true;
    for (uint64_t c = 0; ok && c < std::min<uint64_t>(kSlots, r.chunks); ++c) ok = r.enqueue(c);
    std::thread extra[kMaxThreads - 1];
    uint32_t n = 0;
    const uint32_t want = ok ? (uint32_t)std::min<uint64_t>(host_threads(), r.chunks) - 1u : 0u;
    try {
        for (; n < want; ++n) extra[n] = std::thread([&r] { r.work(true); });
    } catch (...) {  // no thread, or no memory for one: fewer threads
    }
    if (ok) r.work(false);
    for (uint32_t k = 0; k < n; ++k) extra[k].join();
    // nothing may still be on its way into the stage when it is given back
    const hipError_t e = hipStreamSynchronize(s);
    give_back(st);
    const hipError_t first = (hipError_t)r.error.load();
    return first != hipSuccess ? first : e;
}

}  // namespace ising
