// hip_stub.cpp -- a stand-in for the HIP runtime, so that the library's host
// code runs without a GPU: device memory is host memory, copies happen at once,
// kernels do nothing.  Launches and graph instantiations are counted (stub_*).
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
// host function -> kernel name (filled by other files' constructors)
std::map<const void *, std::string> &names() {
    static std::map<const void *, std::string> m;
    return m;
}
std::map<std::string, long> g_launches;
std::map<std::string, dim3> g_grid;
long g_instantiated = 0;
int g_capturing = 0;
dim3 g_g, g_b;
size_t g_s;
hipStream_t g_st;
template <typename H> hipError_t make(H *h) {
    *h = (H)malloc(8);
    return hipSuccess;
}
}  // namespace

extern "C" {
// launches of the kernels whose mangled names contain `part` since the last stub_reset
long stub_launches(const char *part) {
    long n = 0;
    for (const auto &k : g_launches)
        if (k.first.find(part) != std::string::npos) n += k.second;
    return n;
}
// blocks of the last launch of such a kernel
long stub_blocks(const char *part) {
    for (const auto &k : g_grid)
        if (k.first.find(part) != std::string::npos) return (long)k.second.x * k.second.y * k.second.z;
    return -1;
}
long stub_instantiated() { return g_instantiated; }
void stub_reset() {
    g_launches.clear();
    g_grid.clear();
    g_instantiated = 0;
}
// what hipStreamIsCapturing reports from now on
void stub_capturing(int on) { g_capturing = on; }

void **__hipRegisterFatBinary(const void *) {
    static void *p;
    return &p;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *) {
    names()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
    g_g = g, g_b = b, g_s = s, g_st = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st) {
    *g = g_g, *b = g_b, *s = g_s, *st = g_st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **, size_t, hipStream_t) {
    ++g_launches[names()[f]];
    g_grid[names()[f]] = grid;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    if (n > 0) memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    if (n > 0) memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return make(s); }
hipError_t hipStreamDestroy(hipStream_t s) {
    free(s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
    *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return make(g); }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    ++g_instantiated;
    return make(e);
}
hipError_t hipGraphDestroy(hipGraph_t g) {
    free(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    free(e);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return make(e); }
hipError_t hipEventCreate(hipEvent_t *e) { return make(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    *p = nullptr;
    return hipErrorUnknown;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
}
