// A stand-in for the HIP runtime on the CPU, for tests of the library's host
// code: which calls it makes, in which order, on which streams, and what it does
// when one fails.  Loaded with RTLD_GLOBAL before libpm.so, whose calls then
// resolve here.  Memory is the host's; copies and fills are made, those to the
// host when their stream is waited for, as late as the runtime may make them;
// kernels are logged and not run.  One thread at a time.
//
// Log lines (streams and events by number; stream 0 is the null stream):
//   malloc BYTES | free | copy BYTES STREAM | fill BYTES STREAM | sync STREAM (-1: the device)
//   launch KERNEL GRID BLOCK LDS STREAM | graph STREAM
//   stream+ STREAM | stream- STREAM | record EVENT STREAM | wait STREAM EVENT
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

namespace {

std::string g_log, g_copy;
std::map<const void *, std::string> g_kernels;
std::map<std::string, std::pair<long, hipError_t>> g_fail;  // calls until the one that fails
std::map<void *, size_t> g_blocks;
size_t g_used = 0, g_memory = ~size_t(0);
struct Late {
    intptr_t stream;
    void *to;
    const void *from;
    size_t bytes;
};
std::vector<Late> g_late;  // copies to the host
std::set<intptr_t> g_streams, g_capturing;
intptr_t g_next = 1;
hipError_t g_last = hipSuccess;

intptr_t id(const void *p) { return (intptr_t)p; }

// True where this call of `name` has to fail.
bool fails(const char *name) {
    auto f = g_fail.find(name);
    if (f == g_fail.end() || f->second.first-- != 0) return false;
    g_last = f->second.second;
    g_fail.erase(f);
    return true;
}
hipError_t known(hipStream_t s) {
    return s && !g_streams.count(id(s)) ? g_last = hipErrorInvalidHandle : hipSuccess;
}

// The stream (-1: every one) has been waited for.
void arrive(intptr_t stream) {
    std::vector<Late> rest;
    for (const Late &c : g_late) {
        if (stream == -1 || c.stream == stream) std::memcpy(c.to, c.from, c.bytes);
        else rest.push_back(c);
    }
    g_late.swap(rest);
}

template <class... A>
void line(const char *format, A... a) {
    char buf[1024];
    std::snprintf(buf, sizeof(buf), format, a...);
    g_log += buf;
    g_log += '\n';
}

}  // namespace

#define FAKE_CALL(name, ...)                               \
    do {                                                   \
        if (fails(name)) return g_last;                    \
        __VA_ARGS__;                                       \
        return hipSuccess;                                 \
    } while (0)
#define FAKE_ON(name, stream, ...)                         \
    do {                                                   \
        if (known(stream) != hipSuccess) return g_last;    \
        FAKE_CALL(name, __VA_ARGS__);                      \
    } while (0)

extern "C" {

// ---- for the tests
const char *fake_take_log() {
    g_copy.swap(g_log);
    g_log.clear();
    return g_copy.c_str();
}
// Call number `nth` (0: the next) of `name` fails with `code`.
void fake_fail(const char *name, long nth, int code) { g_fail[name] = {nth, (hipError_t)code}; }
// Device memory in bytes, and what is allocated of it.
void fake_memory(size_t bytes) { g_memory = bytes; }
size_t fake_used() { return g_used; }
// The block allocated last.
void *g_last_block = nullptr;
void *fake_last_block() { return g_last_block; }
void fake_capture(intptr_t stream, int on) {
    if (on) g_capturing.insert(stream);
    else g_capturing.erase(stream);
}
// What hipDeviceReset does to streams.
void fake_device_reset() { g_streams.clear(); }

// ---- the runtime
void **__hipRegisterFatBinary(const void *) {
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
    g_kernels[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
static struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} g_config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    g_config = {grid, block, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
    *grid = g_config.grid;
    *block = g_config.block;
    *lds = g_config.lds;
    *s = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t lds, hipStream_t s) {
    FAKE_ON("hipLaunchKernel", s, line("launch %s %u %u %zu %ld", g_kernels[f].c_str(), grid.x, block.x, lds, id(s)));
}

hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "injected error"; }

hipError_t hipGetDevice(int *d) { FAKE_CALL("hipGetDevice", *d = 0); }
int hipGetStreamDeviceId(hipStream_t) { return 0; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { FAKE_CALL("hipDeviceGetAttribute", *v = 256); }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    FAKE_CALL("hipGetDeviceProperties", *p = hipDeviceProp_tR0600{}; std::strcpy(p->gcnArchName, "fake"));
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
    FAKE_CALL("hipOccupancy", *n = 4);
}
hipError_t hipDeviceSynchronize() { FAKE_CALL("hipDeviceSynchronize", line("sync %d", -1); arrive(-1)); }

hipError_t hipMalloc(void **p, size_t bytes) {
    if (g_used + bytes > g_memory) return g_last = hipErrorOutOfMemory;
    FAKE_CALL("hipMalloc", line("malloc %zu", bytes); *p = std::calloc(bytes + 256, 1); g_blocks[*p] = bytes;
              g_used += bytes; g_last_block = *p);
}
hipError_t hipFree(void *p) {
    if (p && !g_blocks.count(p)) return g_last = hipErrorInvalidValue;
    FAKE_CALL("hipFree", line("%s", "free"); arrive(-1); if (p) g_used -= g_blocks[p]; g_blocks.erase(p); std::free(p));
}
hipError_t hipMemcpyAsync(void *to, const void *from, size_t bytes, hipMemcpyKind kind, hipStream_t s) {
    FAKE_ON("hipMemcpyAsync", s, line("copy %zu %ld", bytes, id(s));
            if (kind == hipMemcpyDeviceToHost) g_late.push_back({id(s), to, from, bytes});
            else std::memcpy(to, from, bytes));
}
hipError_t hipMemsetAsync(void *to, int v, size_t bytes, hipStream_t s) {
    FAKE_ON("hipMemsetAsync", s, line("fill %zu %ld", bytes, id(s)); std::memset(to, v, bytes));
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static char symbol[64];
    FAKE_CALL("hipGetSymbolAddress", *p = symbol);
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    FAKE_CALL("hipStreamCreate", g_streams.insert(g_next); *s = (hipStream_t)g_next; line("stream+ %ld", g_next++));
}
hipError_t hipStreamDestroy(hipStream_t s) {
    FAKE_ON("hipStreamDestroy", s, line("stream- %ld", id(s)); g_streams.erase(id(s)));
}
hipError_t hipStreamQuery(hipStream_t s) { FAKE_ON("hipStreamQuery", s, (void)0); }
hipError_t hipStreamSynchronize(hipStream_t s) { FAKE_ON("hipStreamSynchronize", s, line("sync %ld", id(s)); arrive(id(s))); }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    FAKE_ON("hipStreamWaitEvent", s, line("wait %ld %ld", id(s), id(e)));
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c) {
    FAKE_ON("hipStreamIsCapturing", s,
            *c = g_capturing.count(id(s)) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone);
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    FAKE_ON("hipStreamBeginCapture", s, g_capturing.insert(id(s)));
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
    FAKE_ON("hipStreamEndCapture", s, g_capturing.erase(id(s)); *g = (hipGraph_t)1);
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    FAKE_CALL("hipGraphInstantiate", *e = (hipGraphExec_t)1);
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { FAKE_ON("hipGraphLaunch", s, line("graph %ld", id(s))); }

hipError_t hipEventCreate(hipEvent_t *e) { FAKE_CALL("hipEventCreate", *e = (hipEvent_t)g_next++); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    FAKE_ON("hipEventRecord", s, line("record %ld %ld", id(e), id(s)));
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}

}  // extern "C"
