// Test double of the HIP runtime: kernel launches and asynchronous copies are
// recorded instead of run, and one of them can be made to fail, so that the
// library's real launch code (argument rules, grids, error handling) runs and
// can be checked on a machine without a GPU.  Linked with the host code of
// every product source into a separate test library; the product library never
// contains it.  As in the runtime, a failed launch is seen only through
// hipGetLastError, which hands the error over once.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Call { std::string what; dim3 grid, block; };
std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
std::vector<Call> &calls() { static std::vector<Call> v; return v; }
int g_fail = -1;                       // index of the call that fails
hipError_t g_last = hipSuccess;
struct Config { dim3 grid, block; size_t smem; hipStream_t s; } g_cfg;

hipError_t record(const std::string &what, dim3 grid, dim3 block) {
    const bool bad = (int)calls().size() == g_fail;
    calls().push_back({what, grid, block});
    return bad ? hipErrorLaunchFailure : hipSuccess;
}
}  // namespace

extern "C" {
// ---- for the tests
void fake_reset(int fail_index) { calls().clear(); g_fail = fail_index; g_last = hipSuccess; }
int fake_calls() { return (int)calls().size(); }
const char *fake_call_name(int i) { return calls()[i].what.c_str(); }
void fake_call_grid(int i, unsigned *g) { const dim3 d = calls()[i].grid; g[0] = d.x; g[1] = d.y; g[2] = d.z; }

// ---- the runtime
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    names()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t smem, hipStream_t s) {
    g_cfg = {grid, block, smem, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *smem, hipStream_t *s) {
    *grid = g_cfg.grid; *block = g_cfg.block; *smem = g_cfg.smem; *s = g_cfg.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t, hipStream_t) {
    const hipError_t e = record(names()[f], grid, block);
    if (e != hipSuccess) g_last = e;
    return e;
}
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t hipPeekAtLastError() { return g_last; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t) {
    const hipError_t e = record("memcpy", dim3(1), dim3(1));
    if (e == hipSuccess) std::memcpy(dst, src, n);
    return e;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) { std::memcpy(dst, src, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = nullptr; return hipErrorInvalidSymbol; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "injected error"; }
}
