// The calls of the HIP runtime that creating a sparse handle makes, on a machine without a GPU: device memory is host memory, copies are
// made at once, kernels do not run.  What a kernel would have computed and the host reads back is told beforehand (host_hip_answer).
// Device memory can be limited, and a wait be told to report an error.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

namespace {
std::mutex mu;
std::map<void *, size_t> device, pinned;
size_t live, peak, limit = SIZE_MAX, pinned_live, pinned_peak;
int mallocs, refused;
int fail_sync_from = -1, syncs;   // waits from this one on report an error
std::map<size_t, std::vector<char>> answers;   // by the size of the copy to the host
enum { kSuccess = 0, kOutOfMemory = 2, kUnknown = 999, kDeviceToHost = 2 };
thread_local int last;
int report(int e) { if (e) last = e; return e; }
}  // namespace

extern "C" {
// ---- for the tests
void host_hip_reset(size_t bytes) { std::lock_guard<std::mutex> l(mu); limit = bytes; peak = live; pinned_peak = pinned_live; mallocs = refused = syncs = 0; fail_sync_from = -1; }
void host_hip_fail_waits_from(int k) { fail_sync_from = k; }
void host_hip_answer(size_t bytes, const void *data) { answers[bytes].assign((const char *)data, (const char *)data + bytes); }
size_t host_hip_live() { return live; }
size_t host_hip_peak() { return peak; }
size_t host_hip_pinned_live() { return pinned_live; }
size_t host_hip_pinned_peak() { return pinned_peak; }
int host_hip_refused() { return refused; }
int host_hip_syncs() { return syncs; }

// ---- memory
int hipMalloc(void **p, size_t bytes)
{
    std::lock_guard<std::mutex> l(mu);
    ++mallocs;
    *p = nullptr;
    if (bytes > limit || live > limit - bytes) { ++refused; return report(kOutOfMemory); }
    *p = std::calloc(bytes ? bytes : 1, 1);
    device[*p] = bytes;
    live += bytes;
    if (live > peak) peak = live;
    return kSuccess;
}
int hipFree(void *p)
{
    std::lock_guard<std::mutex> l(mu);
    if (!p) return kSuccess;
    auto it = device.find(p);
    if (it == device.end()) std::abort();
    live -= it->second;
    device.erase(it);
    std::free(p);
    return kSuccess;
}
int hipHostMalloc(void **p, size_t bytes, unsigned)
{
    std::lock_guard<std::mutex> l(mu);
    *p = std::calloc(bytes ? bytes : 1, 1);
    pinned[*p] = bytes;
    pinned_live += bytes;
    if (pinned_live > pinned_peak) pinned_peak = pinned_live;
    return kSuccess;
}
int hipHostFree(void *p)
{
    std::lock_guard<std::mutex> l(mu);
    if (!p) return kSuccess;
    auto it = pinned.find(p);
    if (it == pinned.end()) std::abort();
    pinned_live -= it->second;
    pinned.erase(it);
    std::free(p);
    return kSuccess;
}
int hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return kSuccess; }
int hipMemcpy(void *dst, const void *src, size_t bytes, int kind)
{
    auto it = answers.find(bytes);
    std::memcpy(dst, kind == kDeviceToHost && it != answers.end() ? it->second.data() : src, bytes);
    return kSuccess;
}
int hipMemcpyAsync(void *dst, const void *src, size_t bytes, int kind, void *) { return hipMemcpy(dst, src, bytes, kind); }
int hipMemset(void *dst, int v, size_t bytes) { std::memset(dst, v, bytes); return kSuccess; }
int hipMemsetAsync(void *dst, int v, size_t bytes, void *) { return hipMemset(dst, v, bytes); }

// ---- waits and errors
int hipStreamSynchronize(void *)
{
    std::lock_guard<std::mutex> l(mu);
    return report(fail_sync_from >= 0 && syncs++ >= fail_sync_from ? kUnknown : kSuccess);
}
int hipStreamQuery(void *) { return kSuccess; }
int hipGetLastError() { const int e = last; last = 0; return e; }
const char *hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : e ? "error" : "no error"; }
int hipEventCreate(void **e) { *e = std::malloc(1); return kSuccess; }
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *e) { std::free(e); return kSuccess; }
int hipEventRecord(void *, void *) { return kSuccess; }
int hipEventSynchronize(void *) { return kSuccess; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0; return kSuccess; }

// ---- device, kernels
int hipGetDeviceCount(int *n) { *n = 1; return kSuccess; }
int hipGetDevice(int *d) { *d = 0; return kSuccess; }
int hipSetDevice(int) { return kSuccess; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return kSuccess; }
int hipExtStreamGetCUMask(void *, uint32_t n, uint32_t *mask) { for (uint32_t i = 0; i < n; ++i) mask[i] = i < 8 ? ~0u : 0u; return kSuccess; }
int hipFuncSetAttribute(const void *, int, int) { return kSuccess; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 2; return kSuccess; }
int hipGetSymbolAddress(void **p, const void *) { *p = nullptr; return kUnknown; }
struct dim3_ { uint32_t x, y, z; };
int hipLaunchKernel(const void *, dim3_, dim3_, void **, size_t, void *) { return kSuccess; }
int __hipPushCallConfiguration(dim3_, dim3_, size_t, void *) { return kSuccess; }
int __hipPopCallConfiguration(dim3_ *grid, dim3_ *block, size_t *lds, void **st)
{
    *grid = *block = dim3_{1, 1, 1};
    *lds = 0;
    *st = nullptr;
    return kSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}
