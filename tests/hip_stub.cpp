// A HIP runtime for tests of the library's host path without a GPU: device
// memory is host memory, launches are recorded by kernel name (and the kernels
// that move the sweep counter are carried out), and a launch can be made to
// fail.  Loaded before the library with its symbols global.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

extern const int stub_attr_cus;      // the runtime's number of that attribute

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Config { Dim3 grid, block; size_t lds; void *stream; };
std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
std::map<void *, size_t> &blocks() { static std::map<void *, size_t> m; return m; }
std::vector<Config> g_config;
std::vector<std::string> g_log;
std::string g_fail;                  // kernels whose name holds this fail to launch
size_t g_bytes = 0;
int g_error = 0;
}  // namespace

extern "C" {
// for the test
void stub_fail(const char *name) { g_fail = name; }
size_t stub_bytes() { return g_bytes; }
const char *stub_log() {             // kernel names since the last call, one a line
    static std::string out;
    out.clear();
    for (const std::string &s : g_log) out += s + "\n";
    g_log.clear();
    return out.c_str();
}

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, int, void *, void *, void *, void *,
                           int *) { names()[host] = name; }
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t l, void *s) { g_config.push_back({g, b, l, s}); return 0; }
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *l, void **s) {
    const Config c = g_config.back();
    g_config.pop_back();
    *g = c.grid; *b = c.block; *l = c.lds; *s = c.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3, Dim3, void **args, size_t, void *) {
    const std::string &n = names()[f];
    g_log.push_back(n);
    if (!g_fail.empty() && n.find(g_fail) != std::string::npos) return g_error = 719;
    auto ptr = [&](int i) { return *static_cast<int64_t **>(args[i]); };
    auto val = [&](int i) { return *static_cast<int64_t *>(args[i]); };
    if (n.find("begin_run_kernel") != std::string::npos) { *ptr(2) = *ptr(1); *ptr(1) += val(3); }
    if (n.find("restore_t_kernel") != std::string::npos) *ptr(0) = *ptr(1);
    if (n.find("advance_t_kernel") != std::string::npos) *ptr(0) += val(1);
    return 0;
}
int hipGetLastError() { const int e = g_error; g_error = 0; return e; }
const char *hipGetErrorString(int) { return "stub"; }
int hipMalloc(void **p, size_t n) { *p = calloc(1, n ? n : 1); blocks()[*p] = n; g_bytes += n; return *p ? 0 : 2; }
int hipFree(void *p) { if (p) { g_bytes -= blocks()[p]; blocks().erase(p); free(p); } return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { memcpy(d, s, n); return 0; }
int hipGetSymbolAddress(void **p, const void *) { static void *m = calloc(1, 16 << 20); *p = m; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void *) { return 0; }
// compute units, else LDS bytes per workgroup (the library asks for nothing else)
int hipDeviceGetAttribute(int *v, int attr, int) { *v = attr == stub_attr_cus ? 256 : 160 * 1024; return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int threads, size_t lds) {
    *n = std::min<int>(1024 / threads, (int)((160 * 1024) / std::max<size_t>(lds, 1)));
    return 0;
}
int hipEventCreate(void **e) { *e = nullptr; return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = nullptr; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.0f; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = nullptr; return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { *g = nullptr; return 0; }
int hipGraphInstantiate(void **, void *, void **, char *, size_t) { return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipGraphLaunch(void *, void *) { return 0; }
}
