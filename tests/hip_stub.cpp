// A stand-in for the HIP runtime calls that libspx makes, for tests of its
// host code on a machine without a GPU: device memory is host memory, a
// launch is only written down, and allocations, launches and capture can be
// made to fail. Loaded with RTLD_GLOBAL before libspx, whose references then
// bind to it. Kernels do not run, except that the ones that publish a total to
// the host store the next of the totals given.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <string>

namespace {
constexpr int kOk = 0, kOutOfMemory = 2, kLaunchFailure = 719, kCaptureUnsupported = 900;
struct Dim3 { uint32_t x, y, z; };
struct Config { Dim3 grid, block; size_t lds; void* stream; };
struct Counters { void* count; void* clear; uint32_t* done; volatile uint64_t* host; };

std::map<const void*, std::string> g_names;
Config g_config;
std::string g_log;
std::string g_fail_launch;       // a kernel whose launch fails once,
int g_fail_skip = 0;             // after this many that do not
int g_capturing = 0;             // 1: allocation is refused, 2: allowed
size_t g_fail_from = SIZE_MAX, g_fail_to = 0;  // allocations of these sizes fail
int g_error = kOk;
std::deque<uint64_t> g_totals;

void log(const std::string& what) { g_log += what + "\n"; }

int alloc(void** p, size_t bytes) {
    if (g_capturing == 1) return kCaptureUnsupported;
    if (bytes >= g_fail_from && bytes <= g_fail_to) {
        log("malloc-failed " + std::to_string(bytes));
        return g_error = kOutOfMemory;
    }
    log("malloc " + std::to_string(bytes));
    *p = calloc(1, bytes ? bytes : 1);
    return kOk;
}
int copy(void* d, const void* s, size_t n) {
    memmove(d, s, n);
    return kOk;
}
}  // namespace

extern "C" {
void* __hipRegisterFatBinary(const void*) { return &g_config; }
void __hipUnregisterFatBinary(void*) {}
void __hipRegisterFunction(void*, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    g_names[host] = name;
}
void __hipRegisterVar(void*, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    g_config = Config{grid, block, lds, stream};
    return kOk;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = g_config.grid;
    *block = g_config.block;
    *lds = g_config.lds;
    *stream = g_config.stream;
    return kOk;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*) {
    const std::string& name = g_names[f];
    log("launch " + name);
    if (!g_fail_launch.empty() && name.find(g_fail_launch) != std::string::npos && g_fail_skip-- == 0) {
        g_fail_launch.clear();
        return g_error = kLaunchFailure;
    }
    int at = -1;  // of the Counters argument
    if (name.find("k_bfs_seed") != std::string::npos) at = 6;
    if (name.find("k_bfs_update") != std::string::npos) at = 7;
    if (name.find("k_bfs_pull") != std::string::npos) at = 9;
    if (name.find("k_pr_select") != std::string::npos) at = 14;
    if (at >= 0 && !g_totals.empty()) {
        *((Counters*)args[at])->host = g_totals.front();
        g_totals.pop_front();
    }
    return kOk;
}
int hipGetLastError() {
    const int e = g_error;
    g_error = kOk;
    return e;
}
const char* hipGetErrorString(int) { return "stub"; }
int hipMalloc(void** p, size_t n) { return alloc(p, n); }
int hipMallocAsync(void** p, size_t n, void*) { return alloc(p, n); }
int hipHostMalloc(void** p, size_t n, unsigned) { return alloc(p, n); }
int hipFree(void* p) {
    log("free");
    free(p);
    return kOk;
}
int hipFreeAsync(void* p, void*) { return hipFree(p); }
int hipHostFree(void* p) { return hipFree(p); }
int hipMemcpy(void* d, const void* s, size_t n, int) { return copy(d, s, n); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { return copy(d, s, n); }
int hipMemset(void* d, int v, size_t n) { return memset(d, v, n), kOk; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { return memset(d, v, n), kOk; }
int hipStreamSynchronize(void*) {
    log("sync");
    return g_capturing ? kCaptureUnsupported : kOk;
}
int hipDeviceSynchronize() { return hipStreamSynchronize(nullptr); }
int hipStreamIsCapturing(void*, int* status) { return *status = g_capturing ? 1 : 0, kOk; }
int hipStreamGetDevice(void*, int* d) { return *d = 0, kOk; }
int hipGetDevice(int* d) { return *d = 0, kOk; }
int hipSetDevice(int) { return kOk; }
int hipDeviceGetAttribute(int* v, int, int) { return *v = 256, kOk; }
int hipFuncSetAttribute(const void*, int, int) { return kOk; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 2, kOk; }
int hipEventCreate(void** e) { return *e = &g_config, kOk; }
int hipEventDestroy(void*) { return kOk; }
int hipEventRecord(void*, void*) { return kOk; }
int hipEventSynchronize(void*) { return kOk; }
int hipEventElapsedTime(float* t, void*, void*) { return *t = 0, kOk; }
int hipGetSymbolAddress(void** p, const void*) { return *p = nullptr, 1; }

// for the tests
const char* stub_log() { return g_log.c_str(); }
void stub_clear_log() { g_log.clear(); }
void stub_capturing(int mode) { g_capturing = mode; }
void stub_fail_sizes(size_t from, size_t to) {
    g_fail_from = from;
    g_fail_to = to;
}
void stub_fail_launch(const char* kernel, int skip) {
    g_fail_launch = kernel;
    g_fail_skip = skip;
}
void stub_total(uint64_t v) { g_totals.push_back(v); }
}
