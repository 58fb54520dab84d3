// A HIP runtime that runs nothing: loaded ahead of the library in a process of its own, it lets the library's host path run
// without a GPU and fail where a test wants it to.  Device memory is host memory; launches and copies are written down, with the
// arguments that the test asked for.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 { uint32_t x, y, z; };
std::map<const void*, std::string> kernels;                  // host stub -> mangled name
std::vector<std::string> calls;
std::string joined;
std::map<std::string, std::vector<int>> fail;                // call or kernel (part of its name) -> which of the next calls fail
std::map<std::string, int> seen;
std::map<std::string, std::vector<int>> watched;             // kernel (part of its name) -> its int arguments to write down
int last_error = 0;
struct { Dim3 grid, block; size_t shared; void* stream; } config;

bool fails(const std::string& name) {
    for (auto& f : fail) {
        if (name.find(f.first) == std::string::npos) continue;
        const int n = ++seen[f.first];
        for (int k : f.second)
            if (k == n) return true;
    }
    return false;
}
int answer(const char* name) {
    if (!fails(name)) return 0;
    return last_error = 2;                                    // hipErrorOutOfMemory
}
}  // namespace

extern "C" {

void fake_fail(const char* name, int nth) { fail[name].push_back(nth); seen[name] = 0; }
void fake_watch(const char* kernel, int argument) { watched[kernel].push_back(argument); }
void fake_reset() { calls.clear(); fail.clear(); seen.clear(); last_error = 0; }
const char* fake_calls() {
    joined.clear();
    for (auto& c : calls) joined += c + "\n";
    return joined.c_str();
}

void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels[stub] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t sh, void* st) { config = {g, b, sh, st}; return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* sh, void** st) {
    *g = config.grid; *b = config.block; *sh = config.shared; *st = config.stream;
    return 0;
}
int hipLaunchKernel(const void* stub, Dim3 g, Dim3 b, void** args, size_t, void*) {
    const std::string& name = kernels[stub];
    if (fails(name)) return last_error = 719;                 // hipErrorLaunchFailure
    calls.push_back("launch " + name + " " + std::to_string(g.x) + " " + std::to_string(g.y) + " " + std::to_string(b.x));
    for (auto& w : watched)
        if (name.find(w.first) != std::string::npos)
            for (int k : w.second) calls.back() += " " + std::to_string(*static_cast<const int*>(args[k]));
    return 0;
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return e ? "refused by the test" : "no error"; }
int hipMalloc(void** p, size_t n) {
    if (const int e = answer("hipMalloc")) return e;
    calls.push_back("hipMalloc " + std::to_string(n));
    *p = std::malloc(n);
    return 0;
}
int hipFree(void* p) { std::free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) {
    if (const int e = answer("hipHostMalloc")) return e;
    calls.push_back("hipHostMalloc");
    *p = std::calloc(1, n);
    return 0;
}
int hipHostFree(void* p) { std::free(p); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
    if (const int e = answer("hipMemcpyAsync")) return e;
    calls.push_back("hipMemcpyAsync");
    std::memcpy(d, s, n);
    return 0;
}
int hipStreamSynchronize(void*) { calls.push_back("hipStreamSynchronize"); return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipEventCreate(void** e) { *e = std::malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = std::malloc(1); return 0; }
int hipEventDestroy(void* e) { std::free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) {
    calls.push_back("hipStreamCreateWithFlags");
    *s = std::malloc(1);
    return 0;
}
int hipStreamDestroy(void* s) { std::free(s); return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { *g = std::malloc(1); return 0; }
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) { *e = std::malloc(1); return 0; }
int hipGraphDestroy(void* g) { std::free(g); return 0; }
int hipGraphExecDestroy(void* g) { std::free(g); return 0; }
int hipGraphLaunch(void*, void*) { calls.push_back("hipGraphLaunch"); return 0; }

}  // extern "C"
