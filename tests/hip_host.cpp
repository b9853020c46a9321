// CPU stand-in of the HIP calls that the library's host runtime makes, for
// tests of what it allocates and launches: kernels do nothing and are noted by
// name, device memory is address space of a set capacity, streams and events
// are in order by themselves.  Loaded (globally) before libfftdg.so.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<void *, size_t> live;
size_t in_use = 0, capacity = ~(size_t)0;
std::string names;  // mangled kernel names, one a line
}  // namespace

#define API(...) extern "C" __attribute__((visibility("default"))) __VA_ARGS__

API(void host_capacity(size_t n)) { capacity = n; }
API(size_t host_in_use()) { return in_use; }
API(void host_clear()) { names.clear(); }
API(const char *host_launches()) { return names.c_str(); }

API(hipError_t hipMalloc(void **p, size_t n)) {
    *p = nullptr;
    if (n > capacity || in_use > capacity - n) return hipErrorOutOfMemory;
    void *m = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return hipErrorOutOfMemory;
    live[m] = n;
    in_use += n;
    *p = m;
    return hipSuccess;
}
API(hipError_t hipFree(void *p)) {
    if (!p) return hipSuccess;
    const auto it = live.find(p);
    if (it == live.end()) abort();
    munmap(p, it->second);
    in_use -= it->second;
    live.erase(it);
    return hipSuccess;
}
API(hipError_t hipHostMalloc(void **p, size_t n, unsigned)) { return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
API(hipError_t hipHostFree(void *p)) { free(p); return hipSuccess; }
API(hipError_t hipGetSymbolAddress(void **p, const void *)) { static char s[4 << 20]; *p = s; return hipSuccess; }
API(hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)) { memcpy(d, s, n); return hipSuccess; }
API(hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)) { memcpy(d, s, n); return hipSuccess; }
struct Launch {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} next_launch;
API(hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t n, hipStream_t s)) {
    next_launch = Launch{g, b, n, s};
    return hipSuccess;
}
API(hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *n, hipStream_t *s)) {
    *g = next_launch.grid, *b = next_launch.block, *n = next_launch.shared, *s = next_launch.stream;
    return hipSuccess;
}
API(hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, hipStream_t)) {
    if (!g.x || !g.y || !g.z || (size_t)g.x * b.x > 0xffffffffu || g.y > 65535 || g.z > 65535) abort();
    Dl_info i;
    names += dladdr(f, &i) && i.dli_sname ? i.dli_sname : "?";
    names += '\n';
    return hipSuccess;
}
API(hipError_t hipGetDeviceCount(int *n)) { *n = 1; return hipSuccess; }
API(hipError_t hipSetDevice(int)) { return hipSuccess; }
API(hipError_t hipGetLastError()) { return hipSuccess; }
API(hipError_t hipEventCreate(hipEvent_t *e)) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
API(hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)) { return hipEventCreate(e); }
API(hipError_t hipEventDestroy(hipEvent_t e)) { free((void *)e); return hipSuccess; }
API(hipError_t hipEventRecord(hipEvent_t, hipStream_t)) { return hipSuccess; }
API(hipError_t hipEventSynchronize(hipEvent_t)) { return hipSuccess; }
API(hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned)) { return hipSuccess; }
API(hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)) { *s = (hipStream_t)malloc(1); return hipSuccess; }
API(hipError_t hipStreamDestroy(hipStream_t s)) { free((void *)s); return hipSuccess; }
API(hipError_t hipStreamSynchronize(hipStream_t)) { return hipSuccess; }
