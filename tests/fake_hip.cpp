// A stand-in for the HIP runtime in host tests: memory of two GPUs is host memory tagged with a device,
// copies are memcpy, kernels are not run, and every call that touches a GPU is logged with the thread's
// current device.  Loaded before libamr.so, whose references it then satisfies.  Also host memory
// that runs out (on threads other than the one that asks for it) and threads that cannot be started.
#include <hip/hip_runtime_api.h>

#include <dlfcn.h>
#include <malloc.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <system_error>
#include <thread>

namespace {
std::mutex g_mutex;
char g_log[1 << 16];
int g_log_end = 0;
std::map<const char *, std::pair<size_t, int>> g_mem;      // address -> bytes, device
std::map<void *, int> g_streams;
thread_local int g_device = 0;
int g_fail_malloc = 0, g_fail_launch = 0, g_capturing = 0, g_launched = 0, g_pool_device = -1;
uint64_t g_most_blocks = 0;                // of one launch
hipError_t g_error = hipSuccess;
hipStream_t g_stream = nullptr;            // the stream that the call was given
std::atomic<long> g_new_left{-1};          // allocations that worker threads still get; -1: no limit
std::atomic<int> g_threads_left{-1};       // threads that can still be started; -1: no limit
thread_local bool t_main = false;
thread_local dim3 t_grid, t_block;
thread_local size_t t_shared;
thread_local hipStream_t t_stream;

void say(const char *what) {
    std::lock_guard<std::mutex> l(g_mutex);
    const int left = (int)sizeof(g_log) - g_log_end;
    const int n = snprintf(g_log + g_log_end, (size_t)left, "%s %d\n", what, g_device);
    if (n < left) g_log_end += n;
}

int owner(const void *p) {
    std::lock_guard<std::mutex> l(g_mutex);
    auto it = g_mem.upper_bound((const char *)p);
    if (it == g_mem.begin()) return -1;
    --it;
    return (const char *)p < it->first + it->second.first ? it->second.second : -1;
}

void *give(size_t n, int dev) {
    char *p = (char *)aligned_alloc(256, (n + 255) / 256 * 256);
    std::lock_guard<std::mutex> l(g_mutex);
    g_mem[p] = {n, dev};
    return p;
}

void take(void *p) {
    std::lock_guard<std::mutex> l(g_mutex);
    g_mem.erase((const char *)p);
    free(p);
}
// A copy is done when its stream is waited for, as the runtime may; memory that has been freed by then
// has been scribbled over (operator delete below), which its sum shows.
struct Copy {
    void *dst;
    const void *src;
    size_t n;
    uint64_t sum;
    Copy *next;                            // the one enqueued before
} *g_copies = nullptr;

uint64_t sum_of(const void *p, size_t n) {
    uint64_t h = 1469598103934665603ull;
    for (size_t i = 0; i < n; i++) h = (h ^ ((const unsigned char *)p)[i]) * 1099511628211ull;
    return h;
}

void run_copies() {
    Copy *first = nullptr;
    {
        std::lock_guard<std::mutex> l(g_mutex);
        while (g_copies) {                 // in the order in which they were enqueued
            Copy *c = g_copies;
            g_copies = c->next;
            c->next = first;
            first = c;
        }
    }
    while (first) {
        Copy *c = first;
        first = c->next;
        if (sum_of(c->src, c->n) != c->sum) say("source-changed");
        else memcpy(c->dst, c->src, c->n);
        free(c);
    }
}
}  // namespace

extern "C" {

void *fake_alloc(size_t n, int dev) { return give(n, dev); }
void fake_release(void *p) { take(p); }
void fake_stream(void *s, int dev) { g_streams[s] = dev; }
void fake_fail_launch(int on) { g_fail_launch = on; }
void fake_fail_malloc(int on) { g_fail_malloc = on; }
void fake_capturing(int on) { g_capturing = on; }
void fake_call_stream(void *s) { g_stream = (hipStream_t)s; }
void fake_limits(long news, int threads) { t_main = true; g_new_left = news; g_threads_left = threads; }
long fake_held() { return (long)g_mem.size(); }
const char *fake_log() { return g_log; }
void fake_clear() { g_log[g_log_end = 0] = 0, g_most_blocks = 0; }
uint64_t fake_most_blocks() { return g_most_blocks; }

hipError_t hipGetDevice(int *d) { *d = g_device; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    memset(a, 0, sizeof(*a));
    const int d = owner(p);
    if (d < 0) return hipErrorInvalidValue;
    a->type = hipMemoryTypeDevice;
    a->device = d;
    a->devicePointer = (void *)p;
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *d) {
    auto it = g_streams.find((void *)s);
    if (it == g_streams.end()) return hipErrorInvalidHandle;
    *d = it->second;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
    *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMemPoolCreate(hipMemPool_t *m, const hipMemPoolProps *q) {
    g_pool_device = q->location.id;
    *m = (hipMemPool_t)give(1, q->location.id);
    return hipSuccess;
}
hipError_t hipMemPoolDestroy(hipMemPool_t m) { take((void *)m); return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void **p, size_t n, hipMemPool_t, hipStream_t s) {
    if (g_pool_device != g_device) say("pool-elsewhere");
    return hipMallocAsync(p, n, s);
}
// the allocation that fails is counted from 1 (0: none)
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) {
    say("malloc");
    if (g_fail_malloc && --g_fail_malloc == 0) return hipErrorOutOfMemory;
    *p = give(n, g_device);
    return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t) { say("free"); take(p); return hipSuccess; }
// what waits for the whole GPU
hipError_t hipMalloc(void **p, size_t n) { say("malloc-all"); return hipMallocAsync(p, n, nullptr); }
hipError_t hipFree(void *p) { say("free-all"); return hipFreeAsync(p, nullptr); }
hipError_t hipDeviceSynchronize() { say("wait-all"); return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t s) {
    say(s == g_stream ? "copy" : "copy-elsewhere");
    std::lock_guard<std::mutex> l(g_mutex);
    Copy *c = (Copy *)malloc(sizeof(Copy));
    *c = Copy{dst, src, n, sum_of(src, n), g_copies};
    g_copies = c;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { say("stream"); *s = (hipStream_t)0x2000; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
    run_copies();
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = g_launched && g_fail_launch ? hipErrorLaunchFailure : g_error;
    g_error = hipSuccess;
    return e;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
    t_grid = g, t_block = b, t_shared = m, t_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) {
    *g = t_grid, *b = t_block, *m = t_shared, *s = t_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3 g, dim3 b, void **, size_t, hipStream_t) {
    const bool fits = (uint64_t)g.x * b.x < (1ull << 32) && (uint64_t)g.y * b.y < (1ull << 32) &&
                      (uint64_t)g.z * b.z < (1ull << 32) && g.x && g.y && g.z;
    say(fits ? "launch" : "launch-refused");
    g_most_blocks = std::max(g_most_blocks, (uint64_t)g.x * g.y * g.z);
    g_launched = 1;
    g_error = fits ? hipSuccess : hipErrorInvalidConfiguration;
    return g_error;
}
}

void *operator new(size_t n) {
    if (!t_main && g_new_left >= 0 && --g_new_left < 0) {
        g_new_left = 0;
        throw std::bad_alloc();
    }
    void *p = malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept {
    if (p) memset(p, 0xdd, malloc_usable_size(p));
    free(p);
}
void operator delete(void *p, size_t) noexcept { operator delete(p); }

void std::thread::_M_start_thread(_State_ptr state, void (*depend)()) {
    if (g_threads_left >= 0 && --g_threads_left < 0) {
        g_threads_left = 0;
        throw std::system_error(std::make_error_code(std::errc::resource_unavailable_try_again));
    }
    using Start = void (*)(std::thread *, _State_ptr, void (*)());
    static const Start start = (Start)dlsym(RTLD_NEXT, "_ZNSt6thread15_M_start_threadESt10unique_ptrINS_6_StateESt14default_deleteIS1_EEPFvvE");
    start(this, std::move(state), depend);
}
