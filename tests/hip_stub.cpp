// A stand-in for the HIP runtime that runs no kernel and records what the host code enqueues, for the CPU tests of
// libbcsched's launches.  Loaded globally before libbcsched, whose calls then come here.  A launch of 2^32 lanes or
// more along a grid dimension is refused as the runtime refuses it.  Test support; not part of libbcsched.
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

#include <map>
#include <mutex>
#include <string>
#include <vector>

struct dim3 {
    uint32_t x, y, z;
};
typedef void *stream_t;
typedef void *event_t;

namespace {
enum Kind { kLaunch = 0, kMalloc, kFree, kSync, kRecord, kWait };
struct Entry {
    int32_t kind;
    uint64_t stream, pointer, bytes;
    uint32_t grid[3], block[3];
    char name[64];
    uint64_t arg[12];                    // the launch's arguments, as far as the signature of its kernel goes
};
std::mutex g_mutex;
std::vector<Entry> g_log;
std::map<const void *, std::string> g_names;
std::map<std::string, std::string> g_signature;    // a kernel's arguments: '4' or '8' bytes, 'E': 32
uint64_t g_slow_stream = 0;
int g_slow_us = 0, g_last = 0;
uintptr_t g_next_pointer = 0x10000000;
struct Config {
    dim3 grid, block;
    size_t lds;
    stream_t st;
};
thread_local Config t_config;

void add(Kind kind, uint64_t stream, uint64_t pointer, uint64_t bytes) {
    Entry e;
    memset(&e, 0, sizeof e);
    e.kind = kind;
    e.stream = stream;
    e.pointer = pointer;
    e.bytes = bytes;
    std::lock_guard<std::mutex> lock(g_mutex);
    g_log.push_back(e);
}

// the identifier in a mangled name of the anonymous namespace: _ZN12_GLOBAL__N_1<length><identifier>...
std::string plain(const char *mangled) {
    const char *at = strstr(mangled, "_GLOBAL__N_1");
    if (!at) return mangled;
    char *end;
    const long n = strtol(at + strlen("_GLOBAL__N_1"), &end, 10);
    return std::string(end, strnlen(end, (size_t)n));
}
}  // namespace

extern "C" {

void stub_reset() {
    std::lock_guard<std::mutex> lock(g_mutex);
    g_log.clear();
}
int64_t stub_count() {
    std::lock_guard<std::mutex> lock(g_mutex);
    return (int64_t)g_log.size();
}
void stub_get(int64_t i, Entry *out) {
    std::lock_guard<std::mutex> lock(g_mutex);
    *out = g_log[(size_t)i];
}
void stub_signature(const char *kernel, const char *sizes) { g_signature[kernel] = sizes; }
// every launch on this stream takes that long, so that another thread has time to come between
void stub_slow(uint64_t stream, int us) {
    g_slow_stream = stream;
    g_slow_us = us;
}

void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
    g_names[host] = plain(name);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, stream_t st) {
    t_config = Config{grid, block, lds, st};
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, stream_t *st) {
    *grid = t_config.grid;
    *block = t_config.block;
    *lds = t_config.lds;
    *st = t_config.st;
    return 0;
}

int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, stream_t st) {
    if (g_slow_us && (uint64_t)(uintptr_t)st == g_slow_stream) usleep((useconds_t)g_slow_us);
    std::lock_guard<std::mutex> lock(g_mutex);
    const uint32_t g[3] = {grid.x, grid.y, grid.z}, b[3] = {block.x, block.y, block.z};
    for (int d = 0; d < 3; ++d)
        if (g[d] == 0 || b[d] == 0 || (uint64_t)g[d] * b[d] > 0xffffffffull) return g_last = 9;
    Entry e;
    memset(&e, 0, sizeof e);
    e.kind = kLaunch;
    e.stream = (uint64_t)(uintptr_t)st;
    memcpy(e.grid, g, sizeof g);
    memcpy(e.block, b, sizeof b);
    const std::string &name = g_names[f];
    strncpy(e.name, name.c_str(), sizeof e.name - 1);
    const std::string &sizes = g_signature[name];
    size_t at = 0;
    for (size_t i = 0; i < sizes.size(); ++i) {
        const size_t bytes = sizes[i] == 'E' ? 32 : (size_t)(sizes[i] - '0'), words = (bytes + 7) / 8;
        if (at + words > 12) break;
        memcpy(&e.arg[at], args[i], bytes);
        at += words;
    }
    g_log.push_back(e);
    return 0;
}
int hipExtLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, stream_t st, event_t, event_t, int) {
    return hipLaunchKernel(f, grid, block, args, lds, st);
}

int hipGetLastError() {
    const int e = g_last;
    g_last = 0;
    return e;
}
int hipGetDevice(int *dev) {
    *dev = 0;
    return 0;
}
int hipMalloc(void **out, size_t bytes) {
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        *out = (void *)g_next_pointer;
        g_next_pointer += (bytes + 4095) & ~(uintptr_t)4095;
    }
    add(kMalloc, 0, (uint64_t)(uintptr_t)*out, bytes);
    return 0;
}
int hipFree(void *p) {
    add(kFree, 0, (uint64_t)(uintptr_t)p, 0);
    return 0;
}
int hipDeviceSynchronize() {
    add(kSync, 0, 0, 0);
    return 0;
}
int hipEventCreate(event_t *e) {
    *e = malloc(1);
    return 0;
}
int hipEventCreateWithFlags(event_t *e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(event_t e) {
    free(e);
    return 0;
}
int hipEventRecord(event_t, stream_t st) {
    add(kRecord, (uint64_t)(uintptr_t)st, 0, 0);
    return 0;
}
int hipStreamWaitEvent(stream_t st, event_t, unsigned) {
    add(kWait, (uint64_t)(uintptr_t)st, 0, 0);
    return 0;
}
int hipEventQuery(event_t) { return 0; }
int hipEventSynchronize(event_t) { return 0; }
int hipEventElapsedTime(float *ms, event_t, event_t) {
    *ms = 0.f;
    return 0;
}
}
