// The part of the HIP runtime that libflashsplat.so calls, on the host: "device" memory comes from
// calloc under a limit that a test sets, kernels are not run but their names are kept, and a failed
// call's error stays until hipGetLastError reads it. For tests of what the library does on the host
// (test_host_memory.py); loaded before the library, so that its symbols come first.
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {
std::map<const void *, std::string> g_kernels;
std::vector<std::string> g_launched;
std::map<void *, size_t> g_blocks;
size_t g_limit = ~(size_t)0, g_used = 0, g_peak = 0;
thread_local int g_last = 0;
std::mutex g_mu;  // of all the above

int fail(int code) { return g_last = code; }
}  // namespace

struct dim3_t {
    uint32_t x, y, z;
};

extern "C" {

// ---- for the test
void host_limit(size_t bytes) { g_limit = bytes; }
size_t host_used() { return g_used; }
size_t host_peak(int reset)
{
    const size_t p = g_peak;
    if (reset) g_peak = g_used;
    return p;
}
// mangled names of the kernels launched since the last call, one per line
size_t host_launched(char *out, size_t cap)
{
    std::string s;
    for (const std::string &k : g_launched) s += k + "\n";
    g_launched.clear();
    if (s.size() + 1 > cap) return 0;
    memcpy(out, s.c_str(), s.size() + 1);
    return s.size();
}

// ---- kernels
void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    g_kernels[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3_t, dim3_t, size_t, void *) { return 0; }
int __hipPopCallConfiguration(dim3_t *, dim3_t *, size_t *, void **) { return 0; }
int hipLaunchKernel(const void *f, dim3_t, dim3_t, void **, size_t, void *)
{
    std::lock_guard<std::mutex> l(g_mu);
    g_launched.push_back(g_kernels[f]);
    return 0;
}

// ---- memory
int hipMalloc(void **p, size_t bytes)
{
    std::lock_guard<std::mutex> l(g_mu);
    *p = nullptr;
    if (bytes > g_limit || g_used > g_limit - bytes) return fail(2);  // hipErrorOutOfMemory
    *p = calloc(1, bytes ? bytes : 1);
    g_blocks[*p] = bytes;
    g_used += bytes;
    if (g_used > g_peak) g_peak = g_used;
    return 0;
}
int hipFree(void *p)
{
    if (!p) return 0;
    std::lock_guard<std::mutex> l(g_mu);
    const auto it = g_blocks.find(p);
    if (it == g_blocks.end()) return fail(1);
    g_used -= it->second;
    g_blocks.erase(it);
    free(p);
    return 0;
}
int hipHostMalloc(void **p, size_t bytes, unsigned)
{
    *p = calloc(1, bytes);
    return 0;
}
int hipHostFree(void *p)
{
    free(p);
    return 0;
}
int hipMemcpyAsync(void *dst, const void *src, size_t bytes, int, void *)
{
    memcpy(dst, src, bytes);
    return 0;
}
int hipGetSymbolAddress(void **p, const void *)
{
    static void *scratch = calloc(1, 32u << 20);
    *p = scratch;
    return 0;
}

// ---- streams, events, graphs, queries
int hipStreamCreateWithFlags(void **s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamIsCapturing(void *, int *status) { *status = 0; return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { *g = malloc(1); return 0; }
int hipGraphInstantiate(void **x, void *, void *, char *, size_t) { *x = malloc(1); return 0; }
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphDestroy(void *g) { free(g); return 0; }
int hipGraphExecDestroy(void *x) { free(x); return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0.0f; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 4; return 0; }
int hipGetLastError()
{
    const int e = g_last;
    g_last = 0;
    return e;
}
const char *hipGetErrorString(int) { return "error"; }
}
