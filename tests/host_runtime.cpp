// A stand-in for the HIP runtime with which the host code of the library is tested without a GPU (host_lib.py links the
// host halves of csrc/*.hip against it): device memory is host memory, a launch is recorded and, but for the one that copies
// and the one that makes records for the host to go by (host_probe.hip), does nothing.  What can go wrong on the way can be ordered: the n-th allocation on the device or
// on the host fails, or the stream is being captured (then whatever is not allowed meanwhile fails, as in the runtime's
// default capture mode).
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <chrono>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

namespace {

std::mutex g_mutex;
std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> *k = new std::map<const void *, std::string>;
    return *k;
}
std::map<void *, size_t> g_blocks;              // live device blocks
struct Launch { std::string name; int64_t grid, block, lds, filled; };      // (filled: words, of a fill)
std::vector<Launch> g_launches;
std::atomic<int64_t> g_fail_device{-1}, g_fail_new{-1}, g_device_limit{INT64_MAX};
std::atomic<int64_t> g_waits{0}, g_allocs{0}, g_frees{0}, g_device_bytes{0}, g_pinned_bytes{0}, g_new_calls{0}, g_wait_us{0};
std::atomic<int> g_capturing{0}, g_paused{0};
thread_local hipError_t g_last = hipSuccess;
thread_local bool g_inside = false;             // (allocations of the stand-in itself do not fail)
struct Inside { bool was; Inside() : was(g_inside) { g_inside = true; } ~Inside() { g_inside = was; } };

hipError_t result(hipError_t e)
{
    if (e != hipSuccess) g_last = e;
    return e;
}
bool strikes(std::atomic<int64_t> &n) { return n.load() >= 0 && n.fetch_sub(1) == 0; }
void wait_a_little() { if (const int64_t us = g_wait_us.load()) std::this_thread::sleep_for(std::chrono::microseconds(us)); }

}  // namespace

void *operator new(size_t n)
{
    if (!g_inside && !g_paused) {
        ++g_new_calls;
        if (strikes(g_fail_new)) throw std::bad_alloc();
    }
    if (void *p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void *operator new[](size_t n) { return operator new(n); }
void *operator new(size_t n, const std::nothrow_t &) noexcept
{
    try { return operator new(n); } catch (...) { return nullptr; }
}
void operator delete(void *p) noexcept { free(p); }
void operator delete[](void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
void operator delete[](void *p, size_t) noexcept { free(p); }

extern "C" {

// ---- the runtime ----
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    Inside in;
    std::lock_guard<std::mutex> lock(g_mutex);
    kernels()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
static thread_local struct { dim3 grid, block; size_t lds; hipStream_t s; } g_call;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) { g_call = {grid, block, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s)
{
    *grid = g_call.grid; *block = g_call.block; *lds = g_call.lds; *s = g_call.s;
    return hipSuccess;
}

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 0;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
// 160 KB of LDS and sixteen waves a compute unit (what kernels of 128 registers have)
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int threads, size_t lds)
{
    const int by_lds = lds ? (int)((size_t)160 * 1024 / lds) : 32, by_waves = 16 / ((threads + 63) / 64);
    *n = by_lds < by_waves ? by_lds : by_waves;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char room[4096]; *p = room; return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n)
{
    Inside in;
    if (g_capturing) return result(hipErrorStreamCaptureUnsupported);
    *p = nullptr;
    ++g_allocs;
    if ((!g_paused && strikes(g_fail_device)) || (int64_t)n + g_device_bytes.load() > g_device_limit.load()) return result(hipErrorOutOfMemory);
    *p = calloc(1, n);
    std::lock_guard<std::mutex> lock(g_mutex);
    g_blocks[*p] = n;
    g_device_bytes += n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    Inside in;
    if (g_capturing) return result(hipErrorStreamCaptureUnsupported);
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> lock(g_mutex);
    const auto it = g_blocks.find(p);
    if (it == g_blocks.end()) return result(hipErrorInvalidValue);
    g_device_bytes -= it->second;
    g_blocks.erase(it);
    ++g_frees;
    free(p);
    return hipSuccess;
}
static std::map<void *, size_t> g_pinned;
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    Inside in;
    *p = malloc(n);
    std::lock_guard<std::mutex> lock(g_mutex);
    g_pinned[*p] = n;
    g_pinned_bytes += n;
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    Inside in;
    std::lock_guard<std::mutex> lock(g_mutex);
    g_pinned_bytes -= g_pinned[p];
    g_pinned.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    if (g_capturing) return result(hipErrorStreamCaptureUnsupported);
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
// (the caller's stream is the null stream; a stream that the library made is never captured, and waited for on its own)
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = reinterpret_cast<hipStream_t>(&g_waits); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s)
{
    if (g_capturing && !s) return result(hipErrorStreamCaptureUnsupported);
    if (!s) ++g_waits;
    wait_a_little();
    return hipSuccess;
}
hipError_t hipDeviceSynchronize()
{
    if (g_capturing) return result(hipErrorStreamCaptureUnsupported);
    ++g_waits;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c)
{
    *c = g_capturing && !s ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
void host_run_level_records(const void *params);            // (host_probe.hip)
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t)
{
    Inside in;
    std::lock_guard<std::mutex> lock(g_mutex);
    Launch l{kernels()[f], (int64_t)grid.x * grid.y * grid.z, (int64_t)block.x, (int64_t)lds, 0};
    if (l.name.find("copy_in_kernel") != std::string::npos)
        memcpy(*static_cast<void **>(args[2]), *static_cast<void **>(args[1]), (size_t)*static_cast<uint32_t *>(args[0]) * 16);
    if (l.name.find("level_records_kernel") != std::string::npos) host_run_level_records(args[0]);
    if (l.name.find("fill_i32") != std::string::npos) memcpy(&l.filled, args[1], 8);
    if (g_launches.size() < 100000) g_launches.push_back(l);
    return hipSuccess;
}

// ---- what a test orders and reads ----
void host_fail_device(int64_t after) { g_fail_device = after; }          // the allocation after so many more; -1: none
void host_device_limit(int64_t bytes) { g_device_limit = bytes < 0 ? INT64_MAX : bytes; }
void host_fail_new(int64_t after) { g_fail_new = after; }
int64_t host_fail_new_left() { return g_fail_new; }
int64_t host_fail_device_left() { return g_fail_device; }
void host_pause_failures(int on) { g_paused = on; }
void host_capturing(int on) { g_capturing = on; }
void host_slow_copies(int64_t us) { g_wait_us = us; }        // a wait for a stream takes so long
int64_t host_count(const char *what)
{
    const std::string w(what);
    const struct { const char *name; int64_t n; } all[] = {
        {"waits", g_waits}, {"allocs", g_allocs}, {"frees", g_frees}, {"device_bytes", g_device_bytes}, {"pinned_bytes", g_pinned_bytes},
        {"new", g_new_calls}, {"launches", (int64_t)g_launches.size()}};
    for (const auto &c : all)
        if (w == c.name) return c.n;
    return -1;
}
int host_launch(int64_t i, char *name, int64_t room, int64_t *grid, int64_t *block, int64_t *lds, int64_t *filled)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    if (i >= (int64_t)g_launches.size()) return 0;
    const Launch &l = g_launches[i];
    strncpy(name, l.name.c_str(), room - 1);
    name[room - 1] = 0;
    *grid = l.grid; *block = l.block; *lds = l.lds; *filled = l.filled;
    return 1;
}
void host_forget_launches() { std::lock_guard<std::mutex> lock(g_mutex); g_launches.clear(); }

}  // extern "C"
