// A HIP runtime that runs nothing, for the host side of libhough.so: loaded ahead of the library it
// answers the calls the library makes (device memory is host memory) and writes down the kernels that
// would be launched and the order of clears, copies and waits.  tests/test_routes_cpu.py reads it.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void *, std::string> &kernels() {
    static std::map<const void *, std::string> m;
    return m;
}
std::map<const void *, std::string> &vars() {
    static std::map<const void *, std::string> m;
    return m;
}
std::string journal;
size_t largest = ~(size_t)0;      // hipMalloc fails above this
int streams = 0;
struct Call { dim3 grid, block; size_t lds; hipStream_t s; } call;
constexpr size_t kLds = 160 * 1024;

void note(const std::string &line) { journal += line + "\n"; }
// the stream's number (0: the null stream)
int number(hipStream_t s) { return (int)(uintptr_t)s; }
}  // namespace

extern "C" {
const char *fake_journal() { return journal.c_str(); }
void fake_clear() { journal.clear(); }
void fake_largest_malloc(size_t bytes) { largest = bytes; }

void **__hipRegisterFatBinary(const void *) {
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
    kernels()[f] = name;
}
void __hipRegisterVar(void **, void *v, char *, char *name, int, size_t size, int, int) {
    vars()[v] = name;
    (void)size;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
    call = Call{g, b, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
    *g = call.grid; *b = call.block; *lds = call.lds; *s = call.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t s) {
    char line[512];
    std::snprintf(line, sizeof line, "launch %s grid %u,%u block %u lds %zu stream %d", kernels()[f].c_str(), g.x, g.y,
                  b.x, lds, number(s));
    note(line);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static char *scratch = static_cast<char *>(std::calloc(1, 32u << 20));
    *p = scratch;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? (int)kLds : a == hipDeviceAttributeMultiprocessorCount ? 256 : 0;
    return hipSuccess;
}
// Wavefronts a CU holds by registers: what the kernels' launch bounds ask for.
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int threads, size_t lds) {
    const std::string &k = kernels()[f];
    const int waves = threads / 64;
    const bool dense8 = k.find("k_batchILi8ELi1E") != std::string::npos && k.find("ELb0ELb0EE") != std::string::npos;
    const bool wide = waves == 16 || k.find("ELi2E") != std::string::npos || k.find("ELb1EE") != std::string::npos;
    const int by_regs = (dense8 ? 32 : wide ? 16 : 24) / waves;
    const int by_lds = (int)(kLds / (lds + 64));
    *n = by_regs < by_lds ? by_regs : by_lds;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n) {
    *p = n > largest ? nullptr : std::aligned_alloc(256, (n + 256) & ~(size_t)255);
    note((*p ? "malloc " : "refused ") + std::to_string(n));
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n ? n : 1); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);                      // (a blocking call)
    note("copy stream 0");
    note("wait stream 0");
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    note("clear stream 0");
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t s) {
    std::memset(d, v, n);
    note("clear stream " + std::to_string(number(s)));
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = reinterpret_cast<hipStream_t>((uintptr_t)++streams);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    note("wait stream " + std::to_string(number(s)));
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>((uintptr_t)1);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
}
