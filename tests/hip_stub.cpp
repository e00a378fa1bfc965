// hip_stub.cpp -- the HIP runtime calls of the library, on the CPU: device
// memory is host memory, a launch is recorded and runs nothing.  Linked with
// the host side of the library's sources it lets tests follow the C ABI's own
// code without a GPU, also where an allocation fails.
#include "su2_internal.hpp"

#include <hip/hip_ext.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launch {
    std::string name;  // mangled
    unsigned grid[3], block;
    size_t lds;
    int nulls;  // null pointers among the arguments named in ARGS below
    int xcd;    // of a kernel(KArgs, ...): its walk and tile list
    const void *tiles;
};
// registered while the library is loaded, before this file's own objects
std::map<const void *, std::string> &kernels() {
    static std::map<const void *, std::string> m;
    return m;
}
std::vector<Launch> g_launches;
std::map<std::string, std::vector<int>> g_attrs;
long long g_limit = -1, g_countdown = -1, g_room = -1;  // see stub_malloc_limit, _countdown, _room
struct Conf {
    dim3 g, b;
    size_t lds;
    hipStream_t s;
} g_conf;

// pointer arguments that no launch may pass null
struct ArgSet {
    const char *kernel;
    std::vector<int> at;
};
const ArgSet ARGS[] = {{"k_wgauge", {2}}, {"k_wlinks", {1, 5, 6, 7}}, {"k_wloops", {4, 5, 6}}, {"k_wfinal", {0, 2, 3, 4, 5}}};

hipError_t record(const void *f, dim3 g, dim3 b, void **args, size_t lds) {
    Launch l{kernels()[f], {g.x, g.y, g.z}, b.x, lds, 0, -1, nullptr};
    for (const ArgSet &s : ARGS)
        if (l.name.find(s.kernel) != std::string::npos)
            for (int i : s.at) l.nulls += *(void **)args[i] == nullptr;
    if (l.name.find("EvNS_5KArgsE") != std::string::npos) {  // kernel(KArgs, ...)
        const su2::KArgs &a = *(const su2::KArgs *)args[0];
        l.xcd = a.xcd_remap;
        l.tiles = a.tiles;
        l.nulls += !a.desc + !a.tiles + !a.links + !a.st + !a.tries_part;
    }
    g_launches.push_back(l);
    return hipSuccess;
}
}  // namespace

extern "C" {
// Allocations above `bytes` fail (negative: none).
void stub_malloc_limit(long long bytes) { g_limit = bytes; }
// The n-th allocation from now fails, and no other (negative: none).
void stub_malloc_countdown(long long n) { g_countdown = n; }
// Host allocations so far.
int g_host = 0;
int stub_host_mallocs() { return g_host; }
// The next n allocations succeed, later ones do not (negative: all).
void stub_malloc_room(long long n) { g_room = n; }
void stub_clear() { g_launches.clear(); }
int stub_launches() { return (int)g_launches.size(); }
const char *stub_name(int i) { return g_launches[i].name.c_str(); }
int stub_block(int i) { return (int)g_launches[i].block; }
int stub_xcd(int i) { return g_launches[i].xcd; }
const void *stub_tiles(int i) { return g_launches[i].tiles; }
int stub_nulls() {
    int n = 0;
    for (const Launch &l : g_launches) n += l.nulls;
    return n;
}
// Dynamic LDS limits set for the kernels so far: how often one was changed.
int stub_attr_changes() {
    int n = 0;
    for (const auto &a : g_attrs)
        for (size_t i = 1; i < a.second.size(); ++i) n += a.second[i] != a.second[i - 1];
    return n;
}
// Number of kernels given one.
int stub_attrs() { return (int)g_attrs.size(); }

void **__hipRegisterFatBinary(const void *) {
    static void *h = nullptr;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *,
                           int *) {
    kernels()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
    g_conf = Conf{g, b, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
    *g = g_conf.g, *b = g_conf.b, *lds = g_conf.lds, *s = g_conf.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, hipStream_t) {
    return record(f, g, b, args, lds);
}
hipError_t hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, hipStream_t, hipEvent_t,
                              hipEvent_t, int) {
    return record(f, g, b, args, lds);
}
hipError_t hipMalloc(void **p, size_t bytes) {
    *p = nullptr;
    if (g_limit >= 0 && (long long)bytes > g_limit) return hipErrorOutOfMemory;
    if (g_countdown >= 0 && g_countdown-- == 0) return hipErrorOutOfMemory;
    if (g_room == 0) return hipErrorOutOfMemory;
    if (g_room > 0) --g_room;
    *p = std::calloc(1, bytes);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
    ++g_host;
    *p = std::calloc(1, bytes);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) {
    *d = h;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *sym) {
    *p = (void *)sym;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) {
    g_attrs[kernels()[f]].push_back(v);
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
    *n = 4;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    std::memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    *g = (hipGraph_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *e = (hipGraphExec_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
    std::free(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    std::free(e);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
}
