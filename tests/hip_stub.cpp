// A stand-in for the HIP runtime, for tests of the library's host code on machines without a GPU: "device" memory is
// host memory, copies are made at once, kernels are written down and not run.  Loaded with global symbols ahead of the
// library, whose HIP calls then come here.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launch { std::string name; dim3 grid, block; std::vector<void *> arg0; };
struct Range { size_t size; int device; };
std::map<const void *, std::string> g_names;      // host stub of a kernel -> its (mangled) name
std::map<char *, Range> g_memory;                 // what the test calls device memory
std::vector<Launch> g_launches;
struct { dim3 grid, block; size_t shared; hipStream_t stream; } g_config;
int g_fail_at = 0, g_syncs = 0;
hipError_t g_last = hipSuccess;
int *g_pin = nullptr;     // a model's pinned memory, where the one launch of a small model counts itself and says that a wait was given up
bool g_give_up = false;   // whether the next one says so

std::map<char *, Range>::iterator range_of(const void *p)
{
    auto it = g_memory.upper_bound((char *)p);
    if (it == g_memory.begin()) return g_memory.end();
    --it;
    return (char *)p < it->first + it->second.size ? it : g_memory.end();
}
hipError_t error(hipError_t e) { if (e != hipSuccess) g_last = e; return e; }
hipError_t copy(void *dst, const void *src, size_t n)
{
    for (const void *p : {(const void *)dst, src}) {
        auto it = range_of(p);
        if (it != g_memory.end() && (char *)p + n > it->first + it->second.size) return error(hipErrorInvalidValue);
    }
    std::memmove(dst, src, n);
    return hipSuccess;
}
hipError_t launch(const void *f, dim3 grid, dim3 block, void **args)
{
    if (g_fail_at > 0 && --g_fail_at == 0) return error(hipErrorLaunchFailure);
    g_launches.push_back({g_names[f], grid, block, {*(void **)args[0]}});
    // (the one kernel whose answer the library looks at: how many blocks run on each XCD, here all that there are on the third)
    if (std::getenv("STUB_XCD_BLOCKS") && g_names[f].find("xcd_census") != std::string::npos) (*(unsigned **)args[0])[2] = std::atoi(std::getenv("STUB_XCD_BLOCKS"));
    // (... and the one that counts itself there, if it is to run here)
    if (std::getenv("STUB_SMALL_RUNS") && g_names[f].find("small_step") != std::string::npos) {
        ++g_pin[102];
        if (g_give_up) g_pin[100] = 1;
        g_give_up = false;
    }
    return hipSuccess;
}
}  // namespace

extern "C" {
// ---- for the test
void stub_memory(void *p, size_t n, int device) { g_memory[(char *)p] = {n, device}; }
void stub_fail_launch(int nth) { g_fail_at = nth; }       // the nth launch from here on fails (0: none)
void stub_forget(void) { g_launches.clear(); g_syncs = 0; }
void stub_leave_error(void) { g_last = hipErrorInvalidValue; }   // as a call elsewhere in the thread leaves it
void stub_give_up(void) { g_give_up = true; }
int stub_launches(void) { return (int)g_launches.size(); }
int stub_syncs(void) { return g_syncs; }
const char *stub_name(int i) { return g_launches[(size_t)i].name.c_str(); }
unsigned stub_blocks(int i) { const dim3 &g = g_launches[(size_t)i].grid; return g.x * g.y * g.z; }
void *stub_arg0(int i) { return g_launches[(size_t)i].arg0[0]; }

// ---- what the compiler's host code calls
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { g_names[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t st) { g_config = {grid, block, shared, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *st)
{
    *grid = g_config.grid; *block = g_config.block; *shared = g_config.shared; *st = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, hipStream_t) { return launch(f, grid, block, args); }
hipError_t hipLaunchCooperativeKernel(const void *f, dim3 grid, dim3 block, void **args, unsigned, hipStream_t) { return launch(f, grid, block, args); }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 1; return hipSuccess; }

// ---- device, memory, streams
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) { std::memset(p, 0, sizeof(*p)); p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return error(hipErrorInvalidSymbol); }
const char *hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetLastError(void) { hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = std::calloc(1, n);
    if (n == 1024 * sizeof(int)) g_pin = (int *)*p;
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return copy(d, s, n); }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { return copy(d, s, n); }
hipError_t hipStreamSynchronize(hipStream_t) { ++g_syncs; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    auto it = range_of(p);
    if (it == g_memory.end()) return error(hipErrorInvalidValue);
    std::memset(a, 0, sizeof(*a));
    a->type = hipMemoryTypeDevice;
    a->device = it->second.device;
    a->devicePointer = (void *)p;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p)
{
    auto it = range_of(p);
    if (it == g_memory.end()) return error(hipErrorInvalidValue);
    *base = it->first;
    *size = it->second.size;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
}
