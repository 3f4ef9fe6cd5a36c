// The HIP calls that the library makes, on host memory: device memory is
// malloc, copies are memcpy, kernels are counted and not run. Loaded with
// RTLD_GLOBAL before the library (tests/hip_host.py), so that tests without a
// GPU can follow its host side, with failures injected.
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>

namespace {
constexpr int kSuccess = 0, kInvalidValue = 1, kOutOfMemory = 2;
std::mutex mu;
std::map<void*, size_t> device_mem, host_mem;
}  // namespace

extern "C" {

// Counters and switches, read and set by the tests.
long host_fail_malloc = -1;       // this many further device allocations succeed (-1: all)
long host_fail_set_device = -1;   // as above, hipSetDevice
long host_fail_new = -1;          // as above, operator new
long host_live = 0;               // bytes of device memory allocated
std::atomic<long> host_mallocs{0}, host_launches{0}, host_cooperative{0}, host_copies{0};
long host_capturing = 0;           // every stream is being captured
long host_mark = 0;                // cooperative launches set the 4-byte words of pinned memory (time-out marks)

static bool fails(long* left) {
    static std::mutex own;
    std::lock_guard<std::mutex> g(own);
    if (*left < 0) return false;
    if (*left == 0) return true;
    --*left;
    return false;
}

int hipMalloc(void** p, size_t n) {
    ++host_mallocs;
    if (fails(&host_fail_malloc)) return kOutOfMemory;
    *p = calloc(1, n ? n : 1);
    std::lock_guard<std::mutex> g(mu);
    device_mem[*p] = n;
    host_live += (long)n;
    return kSuccess;
}
int hipFree(void* p) {
    if (!p) return kSuccess;
    std::lock_guard<std::mutex> g(mu);
    auto it = device_mem.find(p);
    if (it == device_mem.end()) return kInvalidValue;
    host_live -= (long)it->second;
    device_mem.erase(it);
    free(p);
    return kSuccess;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
    *p = calloc(1, n);
    std::lock_guard<std::mutex> g(mu);
    host_mem[*p] = n;
    return kSuccess;
}
int hipHostFree(void* p) {
    std::lock_guard<std::mutex> g(mu);
    host_mem.erase(p);
    free(p);
    return kSuccess;
}
int hipHostGetDevicePointer(void** d, void* h, unsigned) { return *d = h, kSuccess; }
int hipPointerGetAttributes(int* type, const void* p) {  // the first field
    std::lock_guard<std::mutex> g(mu);
    auto it = host_mem.upper_bound(const_cast<void*>(p));
    if (it == host_mem.begin()) return kInvalidValue;
    --it;
    if ((const char*)p >= (const char*)it->first + it->second) return kInvalidValue;
    return *type = 1, kSuccess;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
    ++host_copies;
    memcpy(d, s, n);
    return kSuccess;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) { return memset(d, v, n), kSuccess; }

int hipGetDevice(int* d) { return *d = 0, kSuccess; }
int hipGetDeviceCount(int* n) { return *n = 1, kSuccess; }
int hipSetDevice(int) { return fails(&host_fail_set_device) ? kInvalidValue : kSuccess; }
int hipDeviceSynchronize() { return kSuccess; }
int hipDeviceGetAttribute(int* v, int, int) { return *v = 256, kSuccess; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 1, kSuccess; }
int hipFuncSetAttribute(const void*, int, int) { return kSuccess; }
int hipGetSymbolAddress(void** p, const void*) {
    static char symbol[1 << 20];
    return *p = symbol, kSuccess;
}
int hipGetLastError() { return kSuccess; }
const char* hipGetErrorName(int) { return "injected"; }

int hipStreamCreateWithFlags(void** s, unsigned) { return *s = malloc(1), kSuccess; }
int hipStreamDestroy(void* s) { return free(s), kSuccess; }
int hipStreamSynchronize(void*) { return kSuccess; }
int hipStreamWaitEvent(void*, void*, unsigned) { return kSuccess; }
int hipStreamIsCapturing(void*, int* v) { return *v = (int)host_capturing, kSuccess; }
int hipStreamBeginCapture(void*, int) { return kSuccess; }
int hipStreamEndCapture(void*, void** g) { return *g = malloc(1), kSuccess; }
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) { return *e = malloc(1), kSuccess; }
int hipGraphLaunch(void*, void*) { return ++host_launches, kSuccess; }
int hipGraphDestroy(void* g) { return free(g), kSuccess; }
int hipGraphExecDestroy(void* e) { return free(e), kSuccess; }
int hipEventCreate(void** e) { return *e = malloc(1), kSuccess; }
int hipEventCreateWithFlags(void** e, unsigned) { return *e = malloc(1), kSuccess; }
int hipEventDestroy(void* e) { return free(e), kSuccess; }
int hipEventRecord(void*, void*) { return kSuccess; }
int hipEventSynchronize(void*) { return kSuccess; }
int hipEventElapsedTime(float* ms, void*, void*) { return *ms = 1.0f, kSuccess; }

struct Dim {
    uint32_t x, y, z;
};
static thread_local Dim cfg_grid, cfg_block;
static thread_local size_t cfg_lds;
static thread_local void* cfg_stream;
int __hipPushCallConfiguration(Dim g, Dim b, size_t lds, void* s) {
    cfg_grid = g, cfg_block = b, cfg_lds = lds, cfg_stream = s;
    return kSuccess;
}
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* lds, void** s) {
    *g = cfg_grid, *b = cfg_block, *lds = cfg_lds, *s = cfg_stream;
    return kSuccess;
}
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void*) { return ++host_launches, kSuccess; }
int hipLaunchCooperativeKernel(const void*, Dim, Dim, void**, unsigned, void*) {
    ++host_cooperative;
    std::lock_guard<std::mutex> g(mu);
    for (auto& m : host_mem)
        if (host_mark && m.second == 4) *(uint32_t*)m.first = 1u;
    return kSuccess;
}

}  // extern "C"

void* operator new(size_t n) {
    if (fails(&host_fail_new)) throw std::bad_alloc();
    if (void* p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
