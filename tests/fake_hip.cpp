// A stand-in for the HIP runtime, for CPU tests of the library's host code: two devices whose memory is host memory,
// launches that are checked against the documented limits and logged instead of run.
//
//   * threads of a launch along a dimension (grid x block) below 2^32, threads of a workgroup at most 1024;
//   * dynamic LDS above 64 KiB only after hipFuncSetAttribute has raised the kernel's limit on the current device.
//
// The log has one line per launch: device, workgroups, threads per workgroup, bytes of dynamic LDS, mangled kernel name.
// A second log says which activations a launch of the per-layer kernels reads and writes, from its arguments: the kernel's name,
// then r or w, address and bytes of each.
#define __HIP_PLATFORM_AMD__ 1
#include "../paper_2306_17266_amd/csrc/kernels.h"
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

namespace {
std::mutex mu;
std::map<const void *, std::string> names;
std::map<const void *, size_t> blocks;
std::map<std::pair<int, const void *>, size_t> lds_limit;
std::map<std::pair<int, std::string>, void *> symbols;
std::map<const void *, std::pair<std::string, size_t>> vars;
std::string log_text;
std::string memory_text;
int element_bytes = 2;
int fail_attributes = 0;
thread_local int device = 0;
thread_local hipError_t last = hipSuccess;
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
};
thread_local Config config;
hipError_t ret(hipError_t e) {
    if (e != hipSuccess) last = e;
    return e;
}
void *take(size_t n) {
    void *p = mmap(nullptr, n ? n : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) return nullptr;
    std::lock_guard<std::mutex> g(mu);
    blocks[p] = n ? n : 1;
    return p;
}
void log_memory(const std::string &name, void **args) {
    using namespace sushi;
    std::string line = name;
    auto add = [&](char how, const void *p, long bytes) {
        char text[64];
        std::snprintf(text, sizeof(text), " %c %llu %ld", how, (unsigned long long)p, bytes);
        if (p) line += text;
    };
    auto has = [&](const char *type) { return name.find(type) != std::string::npos; };
    const long es = element_bytes;
    if (has("8ConvArgs")) {
        const ConvArgs &a = *static_cast<const ConvArgs *>(args[0]);
        const long out = (long)a.B * a.P * a.Q * a.K;
        const bool sums = has("12fc_i8_kernel");  // (reads the pooling's 32-bit sums, writes float32)
        add('r', a.x, (long)a.B * a.H * a.W * a.C * (a.in_f32 || sums ? 4 : es));
        add('r', a.res, out * es);
        add('w', a.y, out * (a.out_f32 || sums ? 4 : es));
        if (has("17conv_small_kernel") || has("16conv_tile_kernel")) add('r', static_cast<const QuantArgs *>(args[2])->gate, (long)a.B * a.C * 4);
    } else if (has("8PoolArgs")) {
        const PoolArgs &a = *static_cast<const PoolArgs *>(args[0]);
        const bool vec = has("10gap_kernel") || has("13gap_i8_kernel");
        add('r', a.x, (long)a.B * a.H * a.W * a.C * es);
        add('r', a.gate, (long)a.B * a.C * 4);
        add('w', a.y, vec ? (long)a.B * a.C * 4 : (long)a.B * a.P * a.Q * a.C * es);
    } else if (has("12ExpandDwArgs")) {
        const ExpandDwArgs &a = *static_cast<const ExpandDwArgs *>(args[0]);
        add('r', a.x, (long)a.B * a.H * a.W * a.C * 2);
        add('w', a.y, (long)a.B * a.P * a.Q * a.K * 2);
        add('w', a.pool, (long)a.B * a.K * static_cast<const ExpandDwGeom *>(args[1])->parts * 4);
    } else if (has("10SeGateArgs")) {
        const SeGateArgs &a = *static_cast<const SeGateArgs *>(args[0]);
        add('r', a.pooled, (long)a.B * a.parts * a.C * 4);
        add('w', a.gate, (long)a.B * a.C * 4);
    }
    memory_text += line + "\n";
}
void give(void *p) {
    std::lock_guard<std::mutex> g(mu);
    auto it = blocks.find(p);
    if (it == blocks.end()) return;
    munmap(p, it->second);
    blocks.erase(it);
}
}  // namespace

extern "C" {
// ---- controls of the tests
const char *fake_log() { return log_text.c_str(); }
const char *fake_memory_log() { return memory_text.c_str(); }
void fake_clear_log() { log_text.clear(), memory_text.clear(); }
void fake_element_bytes(int n) { element_bytes = n; }  // of the activations, for the second log
void fake_fail_attributes(int n) { fail_attributes = n; }  // the next n calls of hipFuncSetAttribute fail

// ---- what the compiler's host code calls
void **__hipRegisterFatBinary(const void *) {
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names[host] = name; }
void __hipRegisterVar(void **, void *host, char *, char *name, int, size_t size, int, int) { vars[host] = {name, size}; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    config = Config{grid, block, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
    *grid = config.grid, *block = config.block, *lds = config.lds, *s = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, hipStream_t) {
    const unsigned long long lim = 1ull << 32;
    if (!g.x || !g.y || !g.z || !b.x || !b.y || !b.z || (unsigned long long)b.x * b.y * b.z > 1024) return ret(hipErrorInvalidConfiguration);
    if ((unsigned long long)g.x * b.x >= lim || (unsigned long long)g.y * b.y >= lim || (unsigned long long)g.z * b.z >= lim)
        return ret(hipErrorInvalidConfiguration);
    std::lock_guard<std::mutex> l(mu);
    if (lds > 65536) {
        auto it = lds_limit.find({device, f});
        if (it == lds_limit.end() || it->second < lds) return ret(hipErrorInvalidValue);
    }
    char line[128];
    std::snprintf(line, sizeof(line), "%d %llu %u %zu ", device, (unsigned long long)g.x * g.y * g.z, b.x * b.y * b.z, lds);
    log_text += line + names[f] + "\n";
    log_memory(names[f], args);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int value) {
    std::lock_guard<std::mutex> l(mu);
    if (fail_attributes > 0) return --fail_attributes, ret(hipErrorNotReady);
    if (value > 160 * 1024) return ret(hipErrorInvalidValue);
    lds_limit[{device, f}] = (size_t)value;
    return hipSuccess;
}

// ---- devices, memory, streams, events
hipError_t hipGetDeviceCount(int *n) { return *n = 2, hipSuccess; }
hipError_t hipSetDevice(int d) { return d < 0 || d > 1 ? ret(hipErrorInvalidDevice) : (device = d, hipSuccess); }
hipError_t hipGetDevice(int *d) { return *d = device, hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t e) {
    static thread_local char text[32];
    std::snprintf(text, sizeof(text), "error %d", (int)e);
    return text;
}
hipError_t hipGetSymbolAddress(void **p, const void *symbol) {
    const auto it = vars.find(symbol);
    if (it == vars.end()) return ret(hipErrorInvalidSymbol);
    void *&m = symbols[{device, it->second.first}];
    if (!m) m = take(it->second.second);
    return *p = m, hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return (*p = take(n)) ? hipSuccess : ret(hipErrorOutOfMemory); }
hipError_t hipFree(void *p) { return give(p), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = reinterpret_cast<hipEvent_t>(&device), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0.f, hipSuccess; }
// (a capture's launches are logged as they are recorded; replays do nothing)
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return *g = reinterpret_cast<hipGraph_t>(&device), hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) { return *x = reinterpret_cast<hipGraphExec_t>(&device), hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
// (not called by what the tests run; the loader asks for them)
hipError_t hipStreamQuery(hipStream_t) { return ret(hipErrorNotSupported); }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return ret(hipErrorNotSupported); }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *, int) { return ret(hipErrorNotSupported); }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *, const void *, int, size_t) { return ret(hipErrorNotSupported); }
}
