// A HIP runtime that launches nothing: it records each kernel's name and grid,
// hands out host memory and fails on request, so that the library's host code runs
// on a machine without a GPU (hip_record.py loads it in front of the real one).
// Read-backs work on host pointers: the copy kernel's words are copied here.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>

namespace {
// The library's allocations fail on request (not those made here).
bool new_fails = false;
int inside = 0;
struct Inside {
    Inside() { ++inside; }
    ~Inside() { --inside; }
};
}  // namespace

void* operator new(std::size_t n) {
    if (new_fails && inside == 0) throw std::bad_alloc();
    return std::malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

namespace {
struct Dim {
    uint32_t x, y, z;
};
std::map<const void*, std::string> names;
std::string calls;
int last_error = 0, launch_error = 0, malloc_error = 0, pointer_device = 0, stream_device = 0, capturing = 0;
Dim g_grid, g_block;
size_t g_shared;
void* g_stream;

void note(const char* what) {
    const Inside in;
    calls += what;
}
int set(int e) {
    if (e) last_error = e;
    return e;
}
int launch(const void* f, Dim g, Dim b, void** args) {
    const Inside in;
    const std::string& name = names[f];
    char line[256];
    std::snprintf(line, sizeof line, "launch %s %u %u %u %u\n", name.c_str(), g.x, g.y, g.z, b.x);
    calls += line;
    if (launch_error) return set(launch_error);
    if (name.find("k_copy_words") != std::string::npos) {
        const uint32_t* src = *static_cast<const uint32_t**>(args[0]);
        uint32_t* dst = *static_cast<uint32_t**>(args[1]);
        std::memcpy(dst, src, 4 * static_cast<size_t>(*static_cast<int*>(args[2])));
    }
    return 0;
}
}  // namespace

extern "C" {
const char* record_calls() { return calls.c_str(); }
void record_clear() { calls.clear(); }
void record_capturing(int on) { capturing = on; }
void record_new_fails(int on) { new_fails = on != 0; }
void record_set(int launch_e, int malloc_e, int pointer_dev, int stream_dev) {
    launch_error = launch_e;
    malloc_error = malloc_e;
    pointer_device = pointer_dev;
    stream_device = stream_dev;
    last_error = 0;
}

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) {
    names[host] = device;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int __hipPushCallConfiguration(Dim g, Dim b, size_t shared, void* stream) {
    g_grid = g;
    g_block = b;
    g_shared = shared;
    g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* shared, void** stream) {
    *g = g_grid;
    *b = g_block;
    *shared = g_shared;
    *stream = g_stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim g, Dim b, void** args, size_t, void*) { return launch(f, g, b, args); }
int hipExtLaunchKernel(const void* f, Dim g, Dim b, void** args, size_t, void*, void*, void*, int) {
    return launch(f, g, b, args);
}
int hipGetLastError() {
    const int e = last_error;
    last_error = 0;
    return e;
}
const char* hipGetErrorString(int) { return "recorded error"; }
int hipHostMalloc(void** p, size_t n, unsigned) {
    note("malloc\n");
    if (malloc_error) return set(malloc_error);
    *p = std::calloc(1, n);
    return 0;
}
int hipHostFree(void* p) {
    note("free\n");
    std::free(p);
    return 0;
}
int hipMemcpy(void* dst, const void* src, size_t n, int) {
    note("memcpy\n");
    std::memcpy(dst, src, n);
    return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int, void*) {
    note("memcpy_async\n");
    std::memcpy(dst, src, n);
    return 0;
}
int hipStreamSynchronize(void*) {
    note("sync\n");
    return set(capturing ? 900 : 0);
}
int hipStreamIsCapturing(void*, int* status) {
    *status = capturing;
    return 0;
}
int hipGetDevice(int* d) {
    *d = stream_device;
    return 0;
}
int hipStreamGetDevice(void*, int* d) {
    *d = stream_device;
    return 0;
}
int hipPointerGetAttribute(void* out, int, void*) {
    *static_cast<int*>(out) = pointer_device;
    return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
    *p = nullptr;
    return set(1);
}
int hipEventCreate(void** e) {
    *e = std::malloc(1);
    return 0;
}
int hipEventDestroy(void* e) {
    std::free(e);
    return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* t, void*, void*) {
    *t = 0.f;
    return 0;
}
}
