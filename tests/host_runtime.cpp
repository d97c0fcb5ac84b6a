// host_runtime.cpp -- the HIP calls and kernel launchers that the library's host
// sources use, replaced by plain memory and a log, so that their choices (which
// launches, what they keep, what they do when memory runs out) are tested
// without a GPU.  "Device" memory is host memory under a settable limit; a
// traversal launch finds one pair per virtual eye and stores none.
#include <hip/hip_runtime_api.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <new>
#include <string>

#include "hrr_types.hpp"

#define EXPORT extern "C" __attribute__((visibility("default")))

using namespace hrr;

namespace {
std::mutex mu;
std::map<void*, size_t> blocks;
size_t limit = ~(size_t)0, used = 0;
std::string log_text;
hipError_t last_error = hipSuccess;
bool fail_device_sync = false;
float spread = 1.0f;
long new_countdown = -1;   // allocations until operator new fails once; < 0: never

void note(const char* fmt, ...) {
    char buf[256];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    std::lock_guard<std::mutex> g(mu);
    log_text += buf;
    log_text += '\n';
}
hipError_t out(hipError_t e) {
    if (e != hipSuccess) last_error = e;
    return e;
}
}  // namespace

void* operator new(size_t n) {
    if (new_countdown >= 0 && new_countdown-- == 0) throw std::bad_alloc();
    void* p = malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

// ---- controls ----
EXPORT void host_limit(size_t bytes) { limit = bytes; }
EXPORT size_t host_used() { return used; }
EXPORT size_t host_blocks() { return blocks.size(); }
EXPORT void host_fail_device_sync(int on) { fail_device_sync = on != 0; }
EXPORT void host_fail_new(long after) { new_countdown = after; }
EXPORT void host_spread(float x) { spread = x; }   // of the hierarchies built from now on
EXPORT int host_last_error() { return (int)last_error; }
EXPORT size_t host_log(char* dst, size_t cap) {   // and clears it
    std::lock_guard<std::mutex> g(mu);
    const size_t n = log_text.size();
    if (dst && cap > n) {
        memcpy(dst, log_text.c_str(), n + 1);
        log_text.clear();
    }
    return n + 1;
}

// ---- HIP ----
extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    std::lock_guard<std::mutex> g(mu);
    *p = nullptr;
    if (n > limit || used > limit - n) return out(hipErrorOutOfMemory);
    *p = calloc(1, n);
    blocks[*p] = n;
    used += n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    std::lock_guard<std::mutex> g(mu);
    if (!p) return hipSuccess;
    auto it = blocks.find(p);
    if (it == blocks.end()) abort();   // freed twice, or never allocated
    used -= it->second;
    blocks.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
    if (k == hipMemcpyDeviceToHost) note("read %zu", n);
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return fail_device_sync ? out(hipErrorStreamCaptureUnsupported) : hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipGetLastError(void) { const hipError_t e = last_error; last_error = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }

// ---- kernel launchers ----
static hipError_t launched(const TravArgs* A) {
    for (uint32_t q = 0; q < A->n_items; ++q) {
        const ItemDesc& D = A->items[q];
        D.counters[CNT_PAIRS] = D.n_virtual;
        D.counters[CNT_STORED] = D.n_virtual < D.capacity ? D.n_virtual : D.capacity;
    }
    return hipGetLastError();
}
hipError_t hrr_launch_traverse(const TravArgs* A, uint32_t epw, uint32_t method, int stats, int weights, uint32_t grid,
                               hipStream_t) {
    note("nodes epw=%u stack=%u method=%u stats=%d weights=%d items=%u tasks=%u grid=%u", epw, A->stack_cap, method, stats,
         weights, A->n_items, A->n_tasks, grid);
    return launched(A);
}
hipError_t hrr_launch_cull(const TravArgs* A, int weights, int dense, uint32_t grid, hipStream_t) {
    note("blocks dense=%d weights=%d items=%u tasks=%u grid=%u", dense, weights, A->n_items, A->n_tasks, grid);
    return launched(A);
}
size_t hrr_trav_lds_per_wave(uint32_t cap, uint32_t) { return (size_t)cap * 8; }
size_t hrr_trav_lds_per_block(uint32_t n_items, size_t per_wave) { return kWavesPerBlock * per_wave + (n_items + 1) * 4; }
hipError_t hrr_traverse_occupancy(uint32_t, uint32_t, int, int, size_t, int* n) { *n = 7; return hipSuccess; }
hipError_t hrr_cull_occupancy(int, int dense, uint32_t, int* n) { *n = dense ? 5 : 8; return hipSuccess; }
hipError_t hrr_launch_order(const OrderItem*, const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t, const uint32_t*,
                            uint32_t, uint32_t*, uint32_t*, uint32_t*, int, hipStream_t) {
    note("order");
    return hipSuccess;
}
hipError_t hrr_launch_compact(const ItemDesc*, uint32_t, uint32_t*, hipStream_t) {
    note("compact");
    return hipSuccess;
}
static unsigned char scratch[kNoAllocScratchBytes];
hipError_t hrr_noalloc_scratch(int, void** p) { *p = scratch; return hipSuccess; }
hipError_t hrr_launch_noalloc_setup(const ItemDesc* D, uint32_t, void* base, hipStream_t) {
    memcpy(static_cast<unsigned char*>(base) + kNoAllocItem, D, sizeof *D);
    return hipSuccess;
}
hipError_t hrr_launch_noalloc_finish(const void*, unsigned long long*, hipStream_t) { return hipSuccess; }
hipError_t hrr_launch_rmq(const uint32_t*, const uint32_t*, const uint32_t*, uint64_t, uint32_t, uint32_t*, uint32_t*,
                          unsigned long long*, int, hipStream_t) {
    return hipSuccess;
}
hipError_t hrr_launch_frontier(const Node*, uint32_t, uint32_t, const float*, float* table, hipStream_t) {
    const uint32_t entries = 1;
    memcpy(table + kFrontierCount, &entries, sizeof entries);
    table[kFrontierSpread] = spread;
    return hipSuccess;
}
hipError_t hrr_launch_blocks(const float*, uint32_t, float*, hipStream_t) { return hipSuccess; }
hipError_t hrr_dev_codes(const float*, uint32_t, const float*, uint64_t*, uint32_t*, uint32_t*, hipStream_t) {
    return hipSuccess;
}
hipError_t hrr_dev_sort(void* temp, size_t* bytes, const uint64_t*, uint64_t*, const uint32_t*, uint32_t*, uint32_t n,
                        hipStream_t) {
    if (!temp) *bytes = (size_t)n * 16;
    return hipSuccess;
}
// the lights in the order given
hipError_t hrr_dev_gather(const float* xyz, const uint32_t*, uint32_t n, float* lights, uint32_t* perm, hipStream_t) {
    for (uint32_t i = 0; i < n; ++i) {
        for (int k = 0; k < 3; ++k) lights[4 * (size_t)i + k] = xyz[3 * (size_t)i + k];
        perm[i] = i;
    }
    return hipSuccess;
}
size_t hrr_dev_nodes_words(uint32_t n) { return 8 * (size_t)n + 64; }
hipError_t hrr_dev_nodes(const uint64_t*, uint32_t n, uint32_t, uint32_t, uint32_t*, uint32_t* counts, hipStream_t) {
    counts[0] = n / 2;   // owners
    return hipSuccess;
}
hipError_t hrr_dev_records(const uint32_t*, uint32_t, const float*, const float*, Node*, hipStream_t) { return hipSuccess; }
}
