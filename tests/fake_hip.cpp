// A stand-in for the HIP runtime, for tests of the library's host code without
// a GPU: device memory is host memory (reserved, not committed), copies are
// checked against the allocations and made, launches are checked against the
// runtime's limits and recorded, and no kernel runs. Loaded globally before
// the library, whose HIP calls then resolve here.
#include <sys/mman.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

enum { kOk = 0, kInvalidValue = 1, kNoMemory = 2, kInvalidConfiguration = 9, kInjected = 719 };
constexpr size_t kPage = 4096;

struct Dim3 {
    uint32_t x, y, z;
};

struct Launch {
    const char* name;
    uint32_t grid[3], block[3];
    uint64_t arg[16];   // the first words of the first argument
    void* stream;
};

std::map<char*, size_t> g_mem;
size_t g_live = 0, g_peak = 0, g_limit = SIZE_MAX;
std::map<const void*, std::string> g_kernels;
std::vector<Launch> g_log;
struct Failure {
    int in, times;   // calls until the first that fails, and how many do
};
std::map<std::string, Failure> g_fail;
uint64_t g_blocks = 0;
bool g_in_flight = false;   // a copy since the last wait
int g_last = kOk;
int g_device = 0;
std::map<void*, int> g_stream_device;

int done(int e)
{
    if (e != kOk) g_last = e;
    return e;
}

bool injected(const char* fn)
{
    const auto it = g_fail.find(fn);
    if (it == g_fail.end()) return false;
    Failure& f = it->second;
    if (--f.in > 0) return false;
    if (--f.times == 0) g_fail.erase(it);
    return true;
}

// The allocation that holds p, or none.
std::map<char*, size_t>::iterator find(const void* p)
{
    auto it = g_mem.upper_bound((char*)p);
    if (it == g_mem.begin()) return g_mem.end();
    --it;
    return (char*)p < it->first + it->second ? it : g_mem.end();
}

bool fits(const void* p, size_t n)
{
    const auto it = find(p);
    return it == g_mem.end() || (size_t)((char*)p - it->first) + n <= it->second;
}

void clear(char* p, size_t n)   // without committing untouched pages
{
    char* a = (char*)(((uintptr_t)p + kPage - 1) / kPage * kPage);
    char* b = (char*)(((uintptr_t)p + n) / kPage * kPage);
    if (a >= b) {
        std::memset(p, 0, n);
        return;
    }
    std::memset(p, 0, a - p);
    madvise(a, b - a, MADV_DONTNEED);
    std::memset(b, 0, p + n - b);
}

struct Config {
    Dim3 grid, block;
    size_t lds;
    void* stream;
};
thread_local Config g_config;

}  // namespace

extern "C" {

// ---- for the tests
void fake_limit(size_t bytes) { g_limit = bytes; }
size_t fake_live() { return g_live; }
size_t fake_peak() { return g_peak; }
void fake_peak_reset() { g_peak = g_live; }
void fake_fail(const char* fn, int nth, int times) { g_fail[fn] = Failure{nth, times}; }
void fake_no_failures() { g_fail.clear(); g_last = kOk; }
void fake_clear() { g_log.clear(); fake_no_failures(); }
int fake_launches() { return (int)g_log.size(); }
const char* fake_name(int i) { return g_log[i].name; }
uint64_t fake_threads(int i, int d) { return (uint64_t)g_log[i].grid[d] * g_log[i].block[d]; }
uint64_t fake_arg(int i, int w) { return g_log[i].arg[w]; }
int fake_in_flight() { return g_in_flight; }
int fake_is_device(uint64_t p) { return find((void*)p) != g_mem.end(); }
void fake_device(int d) { g_device = d; }
void fake_stream_device(void* s, int d) { g_stream_device[s] = d; }

// ---- the runtime
int hipMalloc(void** p, size_t n)
{
    *p = nullptr;
    if (injected("hipMalloc") || n > g_limit || g_live > g_limit - n) return done(kNoMemory);
    const size_t bytes = (n + kPage - 1) / kPage * kPage;
    void* m = mmap(nullptr, bytes ? bytes : kPage, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE,
                   -1, 0);
    if (m == MAP_FAILED) return done(kNoMemory);
    g_mem[(char*)m] = n;
    g_live += n;
    if (g_live > g_peak) g_peak = g_live;
    *p = m;
    return kOk;
}
int hipFree(void* p)
{
    if (!p) return kOk;
    const auto it = g_mem.find((char*)p);
    if (it == g_mem.end()) return done(kInvalidValue);
    g_live -= it->second;
    munmap(p, (it->second + kPage - 1) / kPage * kPage + (it->second ? 0 : kPage));
    g_mem.erase(it);
    return kOk;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*)
{
    if (injected("hipMemcpyAsync")) return done(kInjected);
    if (!fits(d, n) || !fits(s, n)) return done(kInvalidValue);
    std::memmove(d, s, n);
    g_in_flight = true;
    return kOk;
}
int hipMemcpy(void* d, const void* s, size_t n, int k) { return hipMemcpyAsync(d, s, n, k, nullptr); }
int hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int, void*)
{
    for (size_t i = 0; i < h; ++i) std::memmove((char*)d + i * dp, (const char*)s + i * sp, w);
    return kOk;
}
int hipMemsetAsync(void* p, int v, size_t n, void*)
{
    if (!fits(p, n)) return done(kInvalidValue);
    if (v == 0) clear((char*)p, n);
    else std::memset(p, v, n);
    return kOk;
}
int hipMemset(void* p, int v, size_t n) { return hipMemsetAsync(p, v, n, nullptr); }

struct PointerAttributes {
    int type, device;
    void *device_pointer, *host_pointer;
    int managed;
    unsigned flags;
};
int hipPointerGetAttributes(PointerAttributes* a, const void* p)
{
    std::memset(a, 0, sizeof(*a));
    if (find(p) == g_mem.end()) return done(kInvalidValue);
    a->type = 2;   // device memory
    a->device_pointer = (void*)p;
    return kOk;
}
int hipMemGetAddressRange(void** base, size_t* size, void* p)
{
    const auto it = find(p);
    if (it == g_mem.end()) return done(kInvalidValue);
    if (base) *base = it->first;
    if (size) *size = it->second;
    return kOk;
}
int hipGetSymbolAddress(void** p, const void*)
{
    static void* m = nullptr;
    if (!m) {
        const int e = hipMalloc(&m, (size_t)64 << 20);
        if (e != kOk) return e;
    }
    *p = m;
    return kOk;
}

int hipGetDevice(int* d) { *d = g_device; return kOk; }
int hipSetDevice(int d) { g_device = d; return kOk; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return kOk; }
int hipGetDevicePropertiesR0600(void*, int) { return done(kInvalidValue); }
int hipDeviceSynchronize() { return kOk; }
int hipFuncSetAttribute(const void*, int, int) { return kOk; }
const char* hipGetErrorString(int e) { return e == kOk ? "no error" : "error of the stand-in runtime"; }
int hipGetLastError()
{
    const int e = g_last;
    g_last = kOk;
    return e;
}

// Events take the workgroups launched so far as their time.
int hipEventCreate(void** e) { *e = std::calloc(1, 8); return kOk; }
int hipEventDestroy(void* e) { std::free(e); return kOk; }
int hipEventRecord(void* e, void*) { *(uint64_t*)e = g_blocks; return kOk; }
int hipEventSynchronize(void*) { return kOk; }
int hipEventElapsedTime(float* ms, void* a, void* b)
{
    *ms = (float)(*(uint64_t*)b - *(uint64_t*)a) * 1e-3f + 1e-6f;
    return kOk;
}

int hipStreamCreateWithFlags(void** s, unsigned) { *s = std::malloc(8); return kOk; }
int hipStreamDestroy(void* s) { std::free(s); return kOk; }
int hipStreamSynchronize(void*)
{
    g_in_flight = false;
    return kOk;
}
int hipStreamIsCapturing(void*, int* st) { *st = 0; return kOk; }
int hipStreamGetDevice(void* s, int* d)
{
    const auto it = g_stream_device.find(s);
    *d = it == g_stream_device.end() ? g_device : it->second;
    return kOk;
}
int hipStreamBeginCapture(void*, int) { return kOk; }
int hipStreamEndCapture(void*, void** g) { *g = std::malloc(8); return kOk; }
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) { *e = std::malloc(8); return kOk; }
int hipGraphDestroy(void* g) { std::free(g); return kOk; }
int hipGraphExecDestroy(void* e) { std::free(e); return kOk; }
int hipGraphLaunch(void*, void*) { return kOk; }

void** __hipRegisterFatBinary(const void*)
{
    static void* handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*)
{
    g_kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* s)
{
    g_config = Config{g, b, lds, s};
    return kOk;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** s)
{
    *g = g_config.grid;
    *b = g_config.block;
    *lds = g_config.lds;
    *s = g_config.stream;
    return kOk;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void** args, size_t lds, void* s)
{
    if (injected("hipLaunchKernel")) return done(kInjected);
    const uint64_t t[3] = {(uint64_t)g.x * b.x, (uint64_t)g.y * b.y, (uint64_t)g.z * b.z};
    if (!t[0] || !t[1] || !t[2] || t[0] > UINT32_MAX || t[1] > UINT32_MAX || t[2] > UINT32_MAX || g.y > 65535 ||
        g.z > 65535 || b.x * b.y * b.z > 1024 || lds > 160 * 1024)
        return done(kInvalidConfiguration);
    Launch l{g_kernels[f].c_str(), {g.x, g.y, g.z}, {b.x, b.y, b.z}, {}, s};
    std::memcpy(l.arg, args[0], sizeof(uint64_t));
    if (g_kernels[f].find("IndexSearchArgs") != std::string::npos) std::memcpy(l.arg, args[0], sizeof(l.arg));
    g_log.push_back(l);
    g_blocks += (uint64_t)g.x * g.y * g.z;
    return kOk;
}

}  // extern "C"
