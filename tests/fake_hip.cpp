// A HIP runtime of one device in host memory whose kernels do nothing, for
// tests of the library's host code without a GPU (tests/test_plan_memory_cpu.py):
// loaded before the library with global symbols, it takes the calls of the real
// runtime.  It counts allocations and can refuse one of them.
#include <cstdlib>
#include <cstring>
#include <set>

namespace {
std::set<void *> g_live;
long g_count = 0, g_refuse = -1, g_launches = 0;
int g_last = 0;
int ok() { return 0; }

int take(void **p, size_t n)
{
    *p = nullptr;
    if (g_count++ == g_refuse) return g_last = 2;  // hipErrorOutOfMemory
    *p = std::malloc(n ? n : 1);
    g_live.insert(*p);
    return 0;
}

int give(void *p)
{
    if (!p) return 0;
    if (!g_live.erase(p)) std::abort();  // freed twice, or never allocated
    std::free(p);
    return 0;
}
}  // namespace

#define FAKE extern "C" __attribute__((visibility("default")))

FAKE void fake_refuse(long k) { g_count = 0, g_refuse = k; }  // the k-th allocation from now on
FAKE long fake_count() { return g_count; }
FAKE long fake_live() { return (long)g_live.size(); }
FAKE long fake_launches() { return g_launches; }
FAKE int fake_last() { return g_last; }

FAKE int hipMalloc(void **p, size_t n) { return take(p, n); }
FAKE int hipHostMalloc(void **p, size_t n, unsigned) { return take(p, n); }
FAKE int hipFree(void *p) { return give(p); }
FAKE int hipHostFree(void *p) { return give(p); }
FAKE int hipMemcpy(void *d, const void *s, size_t n, int) { return std::memcpy(d, s, n), 0; }
FAKE int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *)
{
    return std::memcpy(d, s, n), 0;
}
FAKE int hipMemsetAsync(void *d, int v, size_t n, void *) { return std::memset(d, v, n), 0; }
struct Dim3 {
    unsigned x, y, z;
};
FAKE int __hipPushCallConfiguration(Dim3, Dim3, size_t, void *) { return ok(); }
FAKE int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *lds, void **s)
{
    *g = *b = Dim3{1, 1, 1};
    *lds = 0;
    *s = nullptr;
    return 0;
}
FAKE int hipLaunchKernel(const void *, ...) { return ++g_launches, 0; }
FAKE int hipGetDeviceCount(int *n) { return *n = 1, 0; }
FAKE int hipGetDevice(int *d) { return *d = 0, 0; }
FAKE int hipSetDevice(int) { return ok(); }
FAKE int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }
FAKE int hipDeviceSynchronize() { return ok(); }
FAKE int hipStreamSynchronize(void *) { return ok(); }
FAKE int hipStreamIsCapturing(void *, int *s) { return *s = 0, 0; }
FAKE int hipGetLastError()
{
    const int e = g_last;
    g_last = 0;
    return e;
}
FAKE const char *hipGetErrorString(int) { return "refused"; }
FAKE int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    return *n = 8, 0;
}
FAKE int hipFuncGetAttributes(void *, const void *) { return 1; }
FAKE int hipFuncSetAttribute(const void *, int, int) { return ok(); }
FAKE int hipGetSymbolAddress(void **p, const void *)
{
    static char word[256];
    return *p = word, 0;
}
FAKE void **__hipRegisterFatBinary(const void *)
{
    static void *h = nullptr;
    return &h;
}
FAKE void __hipRegisterFunction(void **, const void *, char *, const char *, ...) {}
FAKE void __hipRegisterVar(void **, void *, char *, char *, ...) {}
FAKE void __hipUnregisterFatBinary(void **) {}
