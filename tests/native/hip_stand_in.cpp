// Stand-in for the HIP runtime calls that the library makes, for tests of its host logic
// on the CPU: device memory is host memory, a kernel launch only leaves a line in a log
// that the test reads, and the test can make a call fail.  Loaded into the global scope
// before the library, whose references then bind to it.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>

namespace {

std::string g_log;                            // one event a line
std::map<const void*, std::string> g_kernel;  // host stub -> kernel name
std::map<void*, size_t> g_alloc;
int64_t g_live = 0;                // bytes allocated
int64_t g_limit = INT64_MAX;       // most bytes
int g_error = 0;                   // what hipGetLastError returns and forgets
int g_null_capture = 0;            // hipStreamIsCapturing's result for the default stream
const char* g_watch = "";          // calls g_then in the g_watch_at-th launch of this kernel
int g_watch_at = 0;
void (*g_then)() = nullptr;

void event(const std::string& what, const void* stream) {
    g_log += what + " " + std::to_string((uintptr_t)stream) + "\n";
}

}  // namespace

extern "C" {

const char* stand_in_log() { return g_log.c_str(); }
void stand_in_clear() { g_log.clear(); }
int64_t stand_in_live() { return g_live; }
void stand_in_limit(int64_t bytes) { g_limit = bytes; }
void stand_in_null_capture(int error) { g_null_capture = error; }
void stand_in_at_launch(const char* kernel, int nth, void (*then)()) {
    g_watch = strdup(kernel);
    g_watch_at = nth;
    g_then = then;
}

// ---- registration and launch ------------------------------------------------
struct Dim3 {
    uint32_t x, y, z;
};
static Dim3 g_grid, g_block;
static size_t g_shared;
static void* g_stream;
static uint64_t g_threads;  // of the last launch

uint64_t stand_in_threads() { return g_threads; }

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
    g_kernel[stub] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
    g_grid = grid, g_block = block, g_shared = shared, g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
    *grid = g_grid, *block = g_block, *shared = g_shared, *stream = g_stream;
    return 0;
}
int hipLaunchKernel(const void* stub, Dim3 grid, Dim3 block, void**, size_t, void* stream) {
    // threads along a dimension, and workgroups along y and z
    if ((uint64_t)grid.x * block.x >> 32 || grid.y > 65535 || grid.z > 65535)
        return g_error = 9;  // hipErrorInvalidConfiguration
    g_threads = (uint64_t)grid.x * block.x * grid.y * block.y * grid.z * block.z;
    const std::string name = g_kernel.count(stub) ? g_kernel[stub] : "?";
    event("launch " + name, stream);
    if (g_then && name.find(g_watch) != std::string::npos && --g_watch_at == 0) g_then();
    return 0;
}
int hipFuncSetAttribute(const void* stub, int, int value) {
    event("attribute " + (g_kernel.count(stub) ? g_kernel[stub] : "?") + " " + std::to_string(value),
          nullptr);
    return 0;
}

// ---- memory -------------------------------------------------------------------
int hipMalloc(void** p, size_t bytes) {
    if (g_live + (int64_t)bytes > g_limit) return g_error = 2;  // hipErrorOutOfMemory
    *p = calloc(1, std::max<size_t>(bytes, 1));
    g_alloc[*p] = bytes;
    g_live += (int64_t)bytes;
    event("malloc " + std::to_string(bytes), nullptr);
    return 0;
}
int hipFree(void* p) {
    if (!g_alloc.count(p)) return 1;  // hipErrorInvalidValue
    g_live -= (int64_t)g_alloc[p];
    g_alloc.erase(p);
    event("free", nullptr);
    free(p);
    return 0;
}
int hipMemcpy(void* dst, const void* src, size_t bytes, int) {
    memcpy(dst, src, bytes);
    return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int, void*) {
    memcpy(dst, src, bytes);
    return 0;
}
int hipGetSymbolAddress(void**, const void*) { return 1; }

// ---- device, streams, events -----------------------------------------------------
int hipGetDevice(int* dev) {
    *dev = 0;
    return 0;
}
int hipSetDevice(int) { return 0; }
const char* hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error of the stand-in"; }
int hipGetLastError() { return std::exchange(g_error, 0); }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void* stream) {
    event("sync", stream);
    return 0;
}
int hipStreamIsCapturing(void* stream, int* status) {
    *status = 0;
    return stream ? 0 : g_null_capture;
}
int hipEventCreate(void** e) {
    *e = malloc(1);
    return 0;
}
int hipEventDestroy(void* e) {
    free(e);
    return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
    *ms = 0;
    return 0;
}
}
