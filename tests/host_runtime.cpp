// A stand-in for the HIP runtime on a machine without a GPU, for tests of the
// library's host code: memory comes from the host, launches do nothing, and the
// n-th launch, allocation or wait from now can be made to fail.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <set>

namespace {
long long g_launches = 0, g_fail_launch = 0, g_fail_sync = 0;
size_t g_limit = 0, g_largest = 0;  // bytes that one allocation may have (0: any)
std::set<void *> g_live;
hipError_t g_last = hipSuccess;
dim3 g_grid, g_block;
size_t g_lds;
hipStream_t g_stream;
hipError_t set(hipError_t e) {
    if (e != hipSuccess) g_last = e;
    return e;
}
}  // namespace

extern "C" {
// for the tests
long long host_launches() { return g_launches; }
long long host_live() { return (long long)g_live.size(); }
unsigned long long host_largest() { size_t n = g_largest; g_largest = 0; return n; }
void host_fail_launch(long long n) { g_fail_launch = n ? g_launches + n : 0; }
void host_fail_sync(int n) { g_fail_sync = n; }
void host_limit(unsigned long long bytes) { g_limit = bytes; }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, uint3 *, uint3 *, dim3 *, dim3 *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
    g_grid = g, g_block = b, g_lds = lds, g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
    *g = g_grid, *b = g_block, *lds = g_lds, *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) {
    return set(++g_launches == g_fail_launch ? hipErrorLaunchFailure : hipSuccess);
}
hipError_t hipMalloc(void **p, size_t n) {
    g_largest = n > g_largest ? n : g_largest;
    *p = nullptr;
    if ((g_limit && n > g_limit) || !(*p = std::calloc(n ? n : 1, 1))) return set(hipErrorOutOfMemory);
    g_live.insert(*p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipFree(void *p) {
    if (p && !g_live.erase(p)) std::abort();  // freed twice, or never allocated
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipStreamSynchronize(hipStream_t) { return set(g_fail_sync && --g_fail_sync == 0 ? hipErrorUnknown : hipSuccess); }
hipError_t hipDeviceSynchronize() { return hipStreamSynchronize(nullptr); }
hipError_t hipGetLastError() { hipError_t e = g_last; g_last = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t) { return "host runtime"; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : 1;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
#undef hipGetDeviceProperties
#undef hipDeviceProp_t
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    return hipSuccess;
}
}
