// hipMalloc with a limit on the size of one allocation, for tests of what the
// library does where memory runs out; loaded before the HIP runtime, to which
// every other call and every smaller allocation goes.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <link.h>

#include <cstring>

namespace {
size_t g_limit = 0;
int find(dl_phdr_info *info, size_t, void *out) {
    if (!std::strstr(info->dlpi_name, "libamdhip64")) return 0;
    void *lib = dlopen(info->dlpi_name, RTLD_NOLOAD | RTLD_NOW);
    *(void **)out = lib ? dlsym(lib, "hipMalloc") : nullptr;
    return *(void **)out != nullptr;
}
}  // namespace

extern "C" void malloc_limit(unsigned long long bytes) { g_limit = bytes; }
extern "C" hipError_t hipMalloc(void **p, size_t n) {
    static void *real = nullptr;
    if (!real) dl_iterate_phdr(find, &real);
    if (!real || (g_limit && n > g_limit)) return hipErrorOutOfMemory;
    return reinterpret_cast<hipError_t (*)(void **, size_t)>(real)(p, n);
}
