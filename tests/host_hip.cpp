// A stand-in for the HIP runtime on the host, for tests of the library's host
// code without a GPU: preloaded in front of libamdhip64, it serves "device"
// memory from the heap, does copies at once, and records kernel launches by
// name instead of running them.  Memory figures, launch times and failures
// are set by the test through the host_hip_* functions.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

namespace {
// (leaked on purpose: the library unregisters its code objects at exit)
struct State {
    std::mutex mu;
    std::map<const void*, std::string> name;     // kernels by host function
    std::map<void*, size_t> live;                // device memory
    std::vector<std::string> log;                // launches in order
    std::vector<std::pair<std::string, float>> ms;
    std::string last;                            // last launch of a timed kernel
    std::vector<std::string>* capture = nullptr;
    size_t live_bytes = 0, free_bytes = 200ull << 30;
    long long queries = 0, mallocs = 0, fail_malloc = 0, launches = 0, fail_launch = 0;
    long long unwaited = 0;  // launches since the last wait
    int error = 0, device = 0, queried_device = -1;
    bool subtract = false;  // free memory falls with what is allocated
};
State& S() {
    static State* s = new State;
    return *s;
}
long long g_new_until_fail = -1;  // operator new calls until one throws, -1: never
thread_local int g_inside = 0;    // in this file: its own allocations never fail
struct Inside {
    Inside() { ++g_inside; }
    ~Inside() { --g_inside; }
};
bool fails_now() { return g_inside == 0 && g_new_until_fail >= 0 && g_new_until_fail-- == 0; }
int set(int e) {
    if (e) S().error = e;
    return e;
}
struct Dim3 {
    uint32_t x, y, z;
};
}  // namespace

void* operator new(size_t n) {
    if (fails_now()) throw std::bad_alloc();
    void* p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept {
    if (fails_now()) return nullptr;
    return std::malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {

// ---- settings and readings ----
void host_hip_fail_new(long long after) { g_new_until_fail = after; }
long long host_hip_new_left() { return g_new_until_fail; }
void host_hip_free_memory(size_t bytes, int subtract) {
    S().free_bytes = bytes;
    S().subtract = subtract != 0;
}
size_t host_hip_live_bytes() { return S().live_bytes; }
long long host_hip_memory_queries() { return S().queries; }
int host_hip_queried_device() { return S().queried_device; }
void host_hip_current_device(int d) { S().device = d; }
// the n-th allocation (launch) from now on fails, n >= 1
void host_hip_fail_malloc(long long n) { S().fail_malloc = n ? S().mallocs + n : 0; }
void host_hip_fail_launch(long long n) { S().fail_launch = n ? S().launches + n : 0; }
long long host_hip_mallocs() { return S().mallocs; }
long long host_hip_launches() { return S().launches; }
long long host_hip_unwaited() { return S().unwaited; }
// launches whose name holds `part` take `ms`
void host_hip_time(const char* part, float ms) { S().ms.emplace_back(part, ms); }
// the launches since the last call, one name a line
size_t host_hip_log(char* out, size_t cap) {
    std::string all;
    for (const std::string& s : S().log) all += s + "\n";
    S().log.clear();
    const size_t n = all.size() < cap ? all.size() : cap;
    std::memcpy(out, all.data(), n);
    return n;
}

// ---- the runtime ----
void** __hipRegisterFatBinary(const void*) {
    static void* h = nullptr;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device_name, unsigned, void*, void*, void*,
                           void*, int*) {
    S().name[host] = device_name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* sh, void** st) {
    *g = *b = Dim3{1, 1, 1};
    *sh = 0;
    *st = nullptr;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void**, size_t, void*) {
    Inside inside;
    std::lock_guard<std::mutex> lk(S().mu);
    if (++S().launches == S().fail_launch) return set(719);
    const std::string& n = S().name[f];
    if (S().capture) {
        S().capture->push_back(n);
        return 0;
    }
    S().log.push_back(n);
    ++S().unwaited;
    if (n.find("k_sample") != std::string::npos) S().last = n;
    return 0;
}
int hipMalloc(void** p, size_t n) {
    Inside inside;
    std::lock_guard<std::mutex> lk(S().mu);
    *p = nullptr;
    if (++S().mallocs == S().fail_malloc || (S().subtract && S().live_bytes + n > S().free_bytes)) return set(2);
    if (!(*p = std::calloc(n ? n : 1, 1))) return set(2);
    S().live[*p] = n;
    S().live_bytes += n;
    return 0;
}
int hipFree(void* p) {
    Inside inside;
    std::lock_guard<std::mutex> lk(S().mu);
    const auto it = S().live.find(p);
    if (!p) return 0;
    if (it == S().live.end()) std::abort();  // freed twice, or never allocated
    S().live_bytes -= it->second;
    S().live.erase(it);
    std::free(p);
    return 0;
}
int hipMemGetInfo(size_t* f, size_t* t) {
    ++S().queries;
    S().queried_device = S().device;
    *f = S().free_bytes - (S().subtract ? S().live_bytes : 0);
    *t = 288ull << 30;
    return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
    S().unwaited = 0;
    std::memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
    std::memcpy(d, s, n);
    return 0;
}
int hipMemcpyToSymbolAsync(const void*, const void*, size_t, size_t, int, void*) { return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) {
    if (n <= (1u << 20)) std::memset(d, v, n);  // (device memory starts as zeros)
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::calloc(n, 1);
    return 0;
}
int hipHostFree(void* p) {
    std::free(p);
    return 0;
}
int hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = h;
    return 0;
}
int hipGetLastError() {
    const int e = S().error;
    S().error = 0;
    return e;
}
const char* hipGetErrorString(int) { return "set by the test"; }
int hipGetDevice(int* d) {
    *d = S().device;
    return 0;
}
int hipSetDevice(int d) {
    S().device = d;
    return 0;
}
int hipDeviceSynchronize() {
    S().unwaited = 0;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
    *v = 100000;
    return 0;
}
int hipGetDevicePropertiesR0600(void* p, int) {
    // (the library reads the number of compute units only; every field of the
    // 1472 bytes is as good)
    for (int i = 0; i < 1472 / 4; ++i) ((int32_t*)p)[i] = 256;
    return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
    *p = nullptr;
    return 1;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 4;
    return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) {
    *s = std::malloc(1);
    return 0;
}
int hipStreamDestroy(void* s) {
    std::free(s);
    return 0;
}
int hipStreamSynchronize(void*) {
    S().unwaited = 0;
    return 0;
}
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) {
    *e = std::malloc(1);
    return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) {
    *e = std::malloc(1);
    return 0;
}
int hipEventDestroy(void* e) {
    std::free(e);
    return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventQuery(void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
    *ms = 1.0f;
    for (const auto& t : S().ms)
        if (S().last.find(t.first) != std::string::npos) *ms = t.second;
    return 0;
}
int hipStreamBeginCapture(void*, int) {
    Inside inside;
    S().capture = new std::vector<std::string>;
    return 0;
}
int hipStreamEndCapture(void*, void** g) {
    *g = S().capture;
    S().capture = nullptr;
    return 0;
}
int hipGraphInstantiate(void** x, void* g, void*, char*, size_t) {
    Inside inside;
    *x = new std::vector<std::string>(*(std::vector<std::string>*)g);
    return 0;
}
int hipGraphLaunch(void* x, void*) {
    Inside inside;
    for (const std::string& n : *(std::vector<std::string>*)x) {
        S().log.push_back(n);
        if (n.find("k_sample") != std::string::npos) S().last = n;
    }
    return 0;
}
int hipGraphDestroy(void* g) {
    delete (std::vector<std::string>*)g;
    return 0;
}
int hipGraphExecDestroy(void* x) {
    delete (std::vector<std::string>*)x;
    return 0;
}

}  // extern "C"
