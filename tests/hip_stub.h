// A HIP runtime without a GPU for tests of the library's host side: a program that includes this file and links libsj.so defines the
// HIP calls itself, so the library's resolve to these.  Device memory is host memory, kernels do nothing (sj_kv_set_state's sets the
// length), graphs are empty; every call is written to `calls` by name (launches by the kernel's name), and a call can be told to fail.
#include "sj.h"

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

static std::vector<std::string> calls;
static std::string fail_name;          // the fail_nth-th call of this name fails
static int fail_nth = 0;
static void* const CAPTURING = (void*)0x2000;     // a stream that the caller is capturing
static int last_error = 0;
static bool quiet = false;             // keep no record
// (made on first use: the library registers its kernels before this program's own objects exist)
static std::map<const void*, std::string>& kernel_names() { static std::map<const void*, std::string> names; return names; }

static int seen(const char* name) {
    if (quiet) return 0;
    calls.emplace_back(name);
    return last_error = (fail_name == name && --fail_nth == 0) ? 1 : 0;
}
[[maybe_unused]] static void fail_next(const char* name, int nth) { fail_name = name; fail_nth = nth; }
// position of the first call whose name starts so, from `from` on; -1: none
static int first(const char* name, int from = 0) {
    for (size_t i = from; i < calls.size(); ++i)
        if (calls[i].compare(0, std::strlen(name), name) == 0) return (int)i;
    return -1;
}

struct Dim3 { uint32_t x, y, z; };

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* module = nullptr; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernel_names()[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3*, Dim3*, size_t*, void**) { return 0; }
int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*) {
    const std::string& name = kernel_names()[f];
    if (name.find("set_state") != std::string::npos) (*(int32_t**)args[0])[*(int32_t*)args[2]] = *(int32_t*)args[3];      // lengths
    return seen(("launch " + name).c_str());
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "told to fail"; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return seen("hipGetSymbolAddress"); }
int hipMalloc(void** p, size_t n) { *p = std::calloc(1, n); return seen("hipMalloc"); }
int hipFree(void* p) { std::free(p); return seen("hipFree"); }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return seen("hipHostMalloc"); }
int hipHostFree(void* p) { std::free(p); return seen("hipHostFree"); }
int hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return seen("hipMemset"); }
int hipMemsetAsync(void* p, int v, size_t n, void*) { std::memset(p, v, n); return seen("hipMemset"); }
int hipMemcpy(void* d, const void* s, size_t n, int) { std::memcpy(d, s, n); return seen("hipMemcpy"); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { std::memcpy(d, s, n); return seen("hipMemcpy"); }
int hipDeviceSynchronize() { return seen("hipDeviceSynchronize"); }
int hipStreamSynchronize(void*) { return seen("hipStreamSynchronize"); }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = (void*)0x3000; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamBeginCapture(void*, int) { return seen("hipStreamBeginCapture"); }
int hipStreamEndCapture(void*, void** g) { *g = (void*)1; return seen("hipStreamEndCapture"); }
int hipStreamIsCapturing(void* s, int* status) { *status = s == CAPTURING; return 0; }
int hipGraphInstantiate(void** x, void*, void*, char*, size_t) { *x = (void*)1; return seen("hipGraphInstantiate"); }
int hipGraphLaunch(void*, void*) { return seen("hipGraphLaunch"); }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int hipEventCreate(void** e) { *e = (void*)1; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)1; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return seen("hipEventRecord"); }
int hipEventSynchronize(void*) { return seen("hipEventSynchronize"); }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.f; return 0; }
}

// A small model with a cache of 64 positions a sequence, and buffers for its calls
static int failures = 0;
#define CHECK(cond, ...) do { if (!(cond)) { ++failures; std::printf("line %d: ", __LINE__); std::printf(__VA_ARGS__); std::printf("\n"); } } while (0)
struct Small {
    static constexpr int BATCH = 2, GAMMA = 4, VOCAB = 1024, D = 64;
    sj_model* m = nullptr;
    sj_kv* kv = nullptr;
    std::vector<int32_t> tokens = std::vector<int32_t>(256), out = std::vector<int32_t>(256);
    std::vector<float> probs = std::vector<float>(BATCH * 8 * VOCAB), uniforms = std::vector<float>(256), logprob = std::vector<float>(256),
                       hidden = std::vector<float>(BATCH * 8 * D);
    static int fill(void*, int32_t, int32_t, void* dst, size_t n) { std::memset(dst, 0, n); return 0; }
    Small() {
        setenv("SJ_TUNE", "0", 1);
        sj_config c{1, D, 1, 1, 64, 64, VOCAB, SJ_DTYPE_FP32, 10000.f, 1e-5f, 1.f, GAMMA};
        const int32_t cap[BATCH] = {64, 64};
        if (sj_model_load(&c, fill, nullptr, &m) || sj_kv_create(m, BATCH, cap, &kv)) { std::printf("setup: %s\n", sj_last_error()); std::exit(2); }
    }
    ~Small() { sj_kv_free(kv); sj_model_free(m); }
    void lengths(int len) { for (int b = 0; b < BATCH; ++b) sj_kv_set_state(kv, b, len, 1); }
    int step(int gamma, void* st) { return sj_verify_step(m, kv, gamma, tokens.data(), probs.data(), uniforms.data(), 0.5f, out.data(), out.data(), st); }
    int head(int gamma, void* st) { return sj_verify_head(m, kv, gamma, hidden.data(), tokens.data(), probs.data(), uniforms.data(), 0.5f, out.data(), out.data(), st); }
    int draft(int gamma, int feed, void* st) { return sj_draft_block(m, kv, gamma, uniforms.data(), feed, out.data(), probs.data(), st); }
    int score(int n, void* st) { return sj_score_block(m, kv, n, tokens.data(), tokens.data(), logprob.data(), 0, nullptr, st); }
    int prefill(int seq, int n, void* st) { return sj_prefill(m, kv, seq, tokens.data(), n, st); }
};
