// A stand-in for the HIP runtime on a machine without a GPU, for tests of the
// library's host code: device memory is host memory, kernels are recorded by
// name and not run, a stream and an event belong to the device they were made
// on.  Loaded before libtmqcd.so with its symbols global.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

struct Dim3 {
    uint32_t x, y, z;
};
namespace {
std::mutex mu;
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
std::vector<std::string> launches;  // "name x y z"; copies to the host "copy bytes 0 0"
std::set<const void*> pinned;
thread_local int current = 0;
struct Owned {
    int device;
};
thread_local struct {
    Dim3 g, b;
    size_t sh;
    void* st;
} conf;
int device_of(void* stream) { return stream ? ((Owned*)stream)->device : current; }
void* host(size_t n) {
    void* p = nullptr;
    return posix_memalign(&p, 4096, n ? n : 1) ? nullptr : p;
}
}  // namespace

extern "C" {
// ---- for the tests ----
void* standin_stream(int device) { return new Owned{device}; }
int standin_device() { return current; }
int standin_launches() {
    std::lock_guard<std::mutex> l(mu);
    return (int)launches.size();
}
const char* standin_launch(int i) {
    std::lock_guard<std::mutex> l(mu);
    return launches[i].c_str();
}
void standin_clear() {
    std::lock_guard<std::mutex> l(mu);
    launches.clear();
}

// ---- HIP ----
void** __hipRegisterFatBinary(const void*) {
    static void* h;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    int st = 0;
    char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    names()[f] = st == 0 ? d : name;
    free(d);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t sh, void* st) {
    conf = {g, b, sh, st};
    return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* sh, void** st) {
    *g = conf.g;
    *b = conf.b;
    *sh = conf.sh;
    *st = conf.st;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3, void**, size_t, void*) {
    char t[64];
    snprintf(t, sizeof(t), " %u %u %u", g.x, g.y, g.z);
    std::lock_guard<std::mutex> l(mu);
    launches.push_back(names()[f] + t);
    return 0;
}
int hipGetDevice(int* d) {
    *d = current;
    return 0;
}
int hipSetDevice(int d) {
    current = d;
    return 0;
}
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "stand-in error"; }
int hipMalloc(void** p, size_t n) {
    *p = host(n);
    return *p ? 0 : 2;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
    const int e = hipMalloc(p, n);
    std::lock_guard<std::mutex> l(mu);
    pinned.insert(*p);
    return e;
}
int hipPointerGetAttributes(int* type, const void* p) {  // (the type is the first member)
    std::lock_guard<std::mutex> l(mu);
    *type = pinned.count(p) ? 1 : 0;
    return 0;
}
int hipFree(void* p) {
    free(p);
    return 0;
}
int hipHostFree(void* p) {
    std::lock_guard<std::mutex> l(mu);
    pinned.erase(p);
    return hipFree(p);
}
int hipGetSymbolAddress(void** p, const void*) {
    static char scratch[4096];
    *p = scratch;
    return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void*) {
    memcpy(d, s, n);
    if (kind == 2) {
        std::lock_guard<std::mutex> l(mu);
        launches.push_back("copy " + std::to_string(n) + " 0 0");
    }
    return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) {
    memset(d, v, n);
    return 0;
}
int hipStreamSynchronize(void*) { return 0; }
int hipEventCreateWithFlags(void** e, unsigned) {
    *e = new Owned{current};
    return 0;
}
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) {
    delete (Owned*)e;
    return 0;
}
int hipEventRecord(void* e, void* st) { return ((Owned*)e)->device == device_of(st) ? 0 : 400; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
    *ms = 1;
    return 0;
}
int hipStreamBeginCapture(void*, int) { return 801; }
int hipStreamEndCapture(void*, void**) { return 801; }
int hipGraphInstantiate(void**, void*, void*, char*, size_t) { return 801; }
int hipGraphLaunch(void*, void*) { return 801; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
}
