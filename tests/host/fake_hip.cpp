// A HIP runtime that computes nothing, for tests of the library's host logic without a GPU: it keeps
// book of allocations (addresses that nothing reads, an optional limit above which hipMalloc fails) and of
// launches (per kernel name, checked against the launch limits).  Copies to the host deliver zeros, or the
// value of fake_set_host_value.  Loaded with RTLD_GLOBAL before librealq.so, whose HIP calls then come here.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 {
    uint32_t x, y, z;
};
std::map<uintptr_t, size_t> blocks;
std::map<const void*, std::string> names;
std::map<std::string, int64_t> launches;
std::map<std::string, int64_t> copies;
size_t held = 0, peak = 0, limit = SIZE_MAX;
uintptr_t next_addr = 1ull << 40;
double host_value = 0.0;
int last_error = 0, bad_launches = 0, mallocs = 0, capturing = 0;
Dim3 cfg_grid, cfg_block;
size_t cfg_shared;
void* cfg_stream;
}  // namespace

extern "C" {
// ---- the test's side
void fake_reset() {
    launches.clear();
    copies.clear();
    peak = held;
    bad_launches = mallocs = 0;
}
void fake_set_limit(int64_t bytes) { limit = bytes < 0 ? SIZE_MAX : (size_t)bytes; }
void fake_set_host_value(double v) { host_value = v; }
int64_t fake_held() { return (int64_t)held; }
int64_t fake_peak() { return (int64_t)peak; }
int64_t fake_mallocs() { return mallocs; }
void fake_set_capturing(int on) { capturing = on; }
int64_t fake_bad_launches() { return bad_launches; }
int64_t fake_copies() {
    int64_t n = 0;
    for (auto& k : copies) n += k.second;
    return n;
}
// launches of the kernels whose (mangled) name holds `part`
int64_t fake_launches(const char* part) {
    int64_t n = 0;
    for (auto& k : launches)
        if (k.first.find(part) != std::string::npos) n += k.second;
    return n;
}

// ---- the runtime's side
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*,
                           int*) {
    names[host] = device;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
    cfg_grid = grid;
    cfg_block = block;
    cfg_shared = shared;
    cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
    *grid = cfg_grid;
    *block = cfg_block;
    *shared = cfg_shared;
    *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void**, size_t shared, void*) {
    launches[names[f]] += 1;
    auto wide = [](uint32_t blocks, uint32_t threads) { return (uint64_t)blocks * threads > UINT32_MAX; };
    if (!g.x || !g.y || !g.z || (uint64_t)b.x * b.y * b.z > 1024 || wide(g.x, b.x) || wide(g.y, b.y) ||
        wide(g.z, b.z) || g.y > 65535 || g.z > 65535 || shared > 160 * 1024) {
        std::fprintf(stderr, "launch limits: %s grid (%u, %u, %u) block %u\n", names[f].c_str(), g.x, g.y, g.z, b.x);
        ++bad_launches;
        return last_error = 9;  // hipErrorInvalidConfiguration
    }
    return 0;
}
int hipMalloc(void** p, size_t n) {
    *p = nullptr;
    if (capturing) {
        std::fprintf(stderr, "hipMalloc of %zu bytes while capturing\n", n);
        ++mallocs;
        return last_error = 900;  // hipErrorStreamCaptureUnsupported
    }
    if (n > limit - held || held > limit) return last_error = 2;  // hipErrorOutOfMemory
    blocks[next_addr] = n;
    *p = reinterpret_cast<void*>(next_addr);
    next_addr += (n + 0xFFFF) / 0x10000 * 0x10000;
    held += n;
    ++mallocs;
    if (held > peak) peak = held;
    return 0;
}
int hipFree(void* p) {
    auto it = blocks.find(reinterpret_cast<uintptr_t>(p));
    if (it == blocks.end()) return p ? (last_error = 1) : 0;
    held -= it->second;
    blocks.erase(it);
    return 0;
}
int hipMemGetInfo(size_t* free_bytes, size_t* total) {
    const size_t all = limit == SIZE_MAX ? (size_t)288 << 30 : limit;
    *total = all;
    *free_bytes = all > held ? all - held : 0;
    return 0;
}
int hipMemcpyAsync(void* dst, const void*, size_t n, int kind, void*) {
    copies[kind == 2 ? "to_host" : "on_device"] += 1;
    if (kind == 2) {  // device to host
        std::memset(dst, 0, n);
        if (n == sizeof(double)) std::memcpy(dst, &host_value, n);
    }
    return 0;
}
int hipGetLastError() {
    const int e = last_error;
    last_error = 0;
    return e;
}
const char* hipGetErrorString(int e) { return e == 2 ? "out of memory" : e == 9 ? "invalid configuration" : "error"; }
int hipGetDevice(int* d) {
    *d = 0;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
    *v = 256;
    return 0;
}
int hipGetSymbolAddress(void** p, const void* sym) {
    *p = const_cast<void*>(sym);
    return 0;
}
int hipStreamIsCapturing(void*, int* status) {
    *status = capturing;
    return 0;
}
int hipStreamSynchronize(void*) { return capturing ? last_error = 900 : 0; }
int hipEventCreate(void** e) {
    *e = reinterpret_cast<void*>(8);
    return 0;
}
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
    *ms = 0.f;
    return 0;
}
}
