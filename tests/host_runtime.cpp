// A HIP runtime without a device, for tests of the library's host code on the CPU.  It
// stands in for libamdhip64.so.7 in a process of its own: device memory is host memory,
// kernels are recorded and not run, and the null stream is as lazy as the API allows, so
// a fill on it takes place only when something waits for that stream.  Work that reaches
// another stream while such a fill is outstanding, or a stream of another device than the
// memory or the current device, is counted as a violation.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Dim3 {
    uint32_t x, y, z;
};
struct Fill {
    void* p;
    int v;
    size_t n;
};
struct Stream {
    int device;
};
struct Config {
    Dim3 g, b;
    size_t lds;
    void* s;
};

int g_devices = 2;
thread_local int t_device = 0;
thread_local std::vector<Config> t_config;
std::vector<Fill> g_pending;            // fills of the null stream nobody has waited for
std::map<void*, std::pair<size_t, int>> g_mem;  // device memory: bytes, device
size_t g_live = 0, g_peak = 0, g_limit = 0, g_host_live = 0;
long g_fail_in = -1;                    // device allocations until one fails
long g_mallocs = 0, g_frees = 0, g_launches = 0;
std::vector<std::string> g_violations;
std::map<const void*, std::string> g_names;
std::vector<std::string> g_log;         // kernels launched, by name

void violation(const std::string& what) { g_violations.push_back(what); }
void drain() {
    for (const Fill& f : g_pending) std::memset(f.p, f.v, f.n);
    g_pending.clear();
}
void stream_work(void* s, const std::string& what) {
    if (!s) return;  // the null stream keeps its own order
    if (!g_pending.empty()) violation(what + " does not wait for a fill on the null stream");
    if (static_cast<Stream*>(s)->device != t_device)
        violation(what + " on a stream of device " + std::to_string(static_cast<Stream*>(s)->device) + " with device " +
                  std::to_string(t_device) + " current");
}

}  // namespace

extern "C" {

// ------------------------------------------------------------ test controls
void stub_reset() {
    g_violations.clear();
    g_log.clear();
    g_mallocs = g_frees = g_launches = 0;
    g_peak = g_live;
    g_fail_in = -1;
    g_limit = 0;
}
void stub_fail_in(long n) { g_fail_in = n; }         // the n-th device allocation from now on (0: the next) fails
void stub_devices(int n) { g_devices = n; }
void stub_limit(size_t bytes) { g_limit = bytes; }   // device memory there is (0: no limit)
size_t stub_live() { return g_live; }
size_t stub_live_on(int device) {
    size_t n = 0;
    for (const auto& m : g_mem)
        if (m.second.second == device) n += m.second.first;
    return n;
}
size_t stub_peak() { return g_peak; }
size_t stub_host_live() { return g_host_live; }
long stub_mallocs() { return g_mallocs; }
long stub_frees() { return g_frees; }
long stub_launches() { return g_launches; }
long stub_violations() { return long(g_violations.size()); }
const char* stub_violation(long k) { return g_violations[size_t(k)].c_str(); }
long stub_logged() { return long(g_log.size()); }
const char* stub_kernel(long k) { return g_log[size_t(k)].c_str(); }

// ------------------------------------------------------------------ runtime
int hipGetDeviceCount(int* n) { return *n = g_devices, 0; }
int hipGetDevice(int* d) { return *d = t_device, 0; }
int hipSetDevice(int d) {
    if (d < 0 || d >= g_devices) return 101;
    t_device = d;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int) { return *v = 160 * 1024, 0; }
int hipDeviceSynchronize() { return drain(), 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int e) { return e == 0 ? "no error" : e == 2 ? "out of memory" : "error"; }
int hipMemGetInfo(size_t* f, size_t* t) {
    *t = size_t(256) << 30;
    *f = *t - g_live;
    return 0;
}
int hipMalloc(void** p, size_t n) {
    if (g_fail_in == 0) return g_fail_in = -1, 2;
    if (g_fail_in > 0) --g_fail_in;
    if (g_limit && g_live + n > g_limit) return 2;
    *p = std::malloc(n);
    if (!*p) return 2;
    std::memset(*p, 0xA5, n < 4096 ? n : 4096);  // never zero by chance
    g_mem[*p] = {n, t_device};
    g_live += n;
    g_peak = g_live > g_peak ? g_live : g_peak;
    ++g_mallocs;
    return 0;
}
int hipFree(void* p) {
    if (!p) return 0;
    drain();  // waits for the device
    auto it = g_mem.find(p);
    if (it == g_mem.end()) {
        violation("free of memory that is not allocated");
        return 1;
    }
    g_live -= it->second.first;
    g_mem.erase(it);
    ++g_frees;
    std::free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::calloc(1, n + 16);
    std::memcpy(*p, &n, sizeof(n));
    *p = static_cast<char*>(*p) + 16;
    g_host_live += n;
    return 0;
}
int hipHostFree(void* p) {
    if (!p) return 0;
    drain();
    size_t n;
    std::memcpy(&n, static_cast<char*>(p) - 16, sizeof(n));
    g_host_live -= n;
    std::free(static_cast<char*>(p) - 16);
    return 0;
}
int hipMemset(void* p, int v, size_t n) { return g_pending.push_back({p, v, n}), 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) {
    if (!s) return hipMemset(p, v, n);
    stream_work(s, "fill");
    std::memset(p, v, n);
    return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
    drain();
    std::memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void* st) {
    if (!st) drain();
    stream_work(st, "copy");
    std::memcpy(d, s, n);
    return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) { return *s = new Stream{t_device}, 0; }
int hipStreamDestroy(void* s) { return delete static_cast<Stream*>(s), 0; }
int hipStreamSynchronize(void* s) {
    if (!s) drain();
    return 0;
}
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) { return *e = new int(t_device), 0; }
int hipEventDestroy(void* e) { return delete static_cast<int*>(e), 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventQuery(void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { return *ms = 0.01f, 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 1, 0; }
int hipGetSymbolAddress(void** p, const void* sym) { return *p = const_cast<void*>(sym), 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { return *g = std::malloc(1), 0; }
int hipGraphInstantiate(void** x, void*, void*, char*, size_t) { return *x = std::malloc(1), 0; }
int hipGraphDestroy(void* g) { return std::free(g), 0; }
int hipGraphExecDestroy(void* x) { return std::free(x), 0; }
int hipGraphLaunch(void*, void* s) { return stream_work(s, "graph"), 0; }
int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void* s) {
    (void)args;
    const std::string& name = g_names[f];
    stream_work(s, name);
    ++g_launches;
    if (g_log.size() < 100000) g_log.push_back(name);
    return 0;
}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* s) {
    t_config.push_back({g, b, lds, s});
    return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** s) {
    const Config c = t_config.back();
    t_config.pop_back();
    *g = c.g;
    *b = c.b;
    *lds = c.lds;
    *s = c.s;
    return 0;
}
void** __hipRegisterFatBinary(const void*) {
    static void* h = nullptr;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    g_names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

}  // extern "C"
