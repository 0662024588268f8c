// A stand-in for the HIP runtime, so that the host code of libompd runs on a machine without a
// GPU: device memory is host memory within a budget, every copy and fill is checked against the
// allocations, and kernels are counted instead of run (their outputs stay zero: every status is
// "ok" and nothing ever changes, which ends each fixed point after its first round).
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {
std::mutex mu;
std::map<char*, size_t> dev;        // device allocations
size_t live = 0, budget = (size_t)64 << 30;
long violations = 0, allocs = 0, fail_at = -1;
long clock_ms = 0;                  // a kernel takes one millisecond
std::vector<size_t> sizes;          // of every allocation so far
std::string first;
struct Kernel { long launches = 0, items = 0; };
std::map<const void*, std::string> names;
std::map<std::string, Kernel> kernels;
std::map<const void*, std::pair<char*, size_t>> symbols;
std::string events;                 // what the runtime was asked to do, in order

void violate(const std::string& what)
{
    if (!violations++) first = what;
}
// a device address and its bytes lie inside one allocation
bool inside(const void* p, size_t n)
{
    char* c = (char*)p;
    auto it = dev.upper_bound(c);
    if (it != dev.begin()) {
        --it;
        if (c >= it->first && c + n <= it->first + it->second) return true;
        if (c < it->first + it->second) return false;
    }
    for (auto& s : symbols)
        if (s.second.first && c >= s.second.first && c + n <= s.second.first + s.second.second) return true;
    return false;
}
hipError_t copy(void* d, const void* s, size_t n, hipMemcpyKind kind)
{
    std::lock_guard<std::mutex> g(mu);
    char b[96];
    snprintf(b, sizeof b, "copy of %zu bytes outside an allocation", n);
    if ((kind == hipMemcpyHostToDevice || kind == hipMemcpyDeviceToDevice) && !inside(d, n)) {
        violate(std::string(b) + " (to the device)");
        return hipErrorInvalidValue;
    }
    if ((kind == hipMemcpyDeviceToHost || kind == hipMemcpyDeviceToDevice) && !inside(s, n)) {
        violate(std::string(b) + " (from the device)");
        return hipErrorInvalidValue;
    }
    memcpy(d, s, n);
    return hipSuccess;
}
void note(const char* e)
{
    std::lock_guard<std::mutex> g(mu);
    events += e;
    events += ' ';
}
}  // namespace

extern "C" {
// ---- what a test asks ----
void standin_budget(size_t bytes) { budget = bytes; }
void standin_fail_alloc(long k) { fail_at = k < 0 ? -1 : allocs + k; }   // the k-th allocation from now fails
size_t standin_live() { return live; }
long standin_allocs() { return allocs; }
size_t standin_alloc_size(long k) { return sizes[k]; }
long standin_violations() { return violations; }
const char* standin_first() { return first.c_str(); }
const char* standin_events() { return events.c_str(); }
void standin_clear_events() { events.clear(); }
static long total(const char* part, bool items)
{
    long t = 0;
    for (auto& k : kernels)
        if (k.first.find(part) != std::string::npos) t += items ? k.second.items : k.second.launches;
    return t;
}
long standin_launches(const char* part) { return total(part, false); }
long standin_items(const char* part) { return total(part, true); }
void standin_clear_kernels() { kernels.clear(); }

// ---- the runtime ----
hipError_t hipMalloc(void** p, size_t n)
{
    std::lock_guard<std::mutex> g(mu);
    sizes.push_back(n);
    if (allocs++ == fail_at || live + n > budget) return hipErrorOutOfMemory;
    char* c = (char*)calloc(1, n ? n : 1);
    dev[c] = n;
    live += n;
    *p = c;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    std::lock_guard<std::mutex> g(mu);
    auto it = dev.find((char*)p);
    if (it == dev.end()) { violate("free of an address that is not an allocation"); return hipErrorInvalidValue; }
    live -= it->second;
    dev.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) { note("memcpy"); return copy(d, s, n, k); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return copy(d, s, n, k); }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t)
{
    std::lock_guard<std::mutex> g(mu);
    if (!inside(d, n)) { violate("fill outside an allocation"); return hipErrorInvalidValue; }
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t)
{
    std::lock_guard<std::mutex> g(mu);
    const std::string& n = names[f];
    Kernel& k = kernels[n];
    ++k.launches;
    ++clock_ms;
    if (n.find("CallTabItem") != std::string::npos) k.items += *(int*)args[1];
    for (const char* part : {"k_nu", "k_ave", "k_mayp", "k_later", "k_live", "k_avf", "k_post", "k_varkind", "k_solve",
                             "k_strip", "k_tin", "k_tmid", "k_tout"})   // (descriptors, tiles or items, ...)
        if (n.find(part) != std::string::npos && !inside(*(void**)args[1], 16)) violate(n + " without its table");
    events += "launch ";
    return hipSuccess;
}
static thread_local dim3 cfg_grid, cfg_block;
static thread_local size_t cfg_shm;
static thread_local hipStream_t cfg_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st)
{
    cfg_grid = g; cfg_block = b; cfg_shm = s; cfg_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st)
{
    *g = cfg_grid; *b = cfg_block; *s = cfg_shm; *st = cfg_stream;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    names[host] = name;
}
void __hipRegisterVar(void**, void* host, char*, char*, int, size_t size, int, int) { symbols[host] = {nullptr, size}; }
hipError_t hipGetSymbolAddress(void** p, const void* s)
{
    auto& y = symbols[s];
    if (!y.first) y.first = (char*)calloc(1, y.second ? y.second : 1);
    *p = y.first;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    p->maxSharedMemoryPerMultiProcessor = 160 * 1024;
    p->sharedMemPerBlock = 64 * 1024;
    p->totalGlobalMem = budget;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }
hipError_t hipDeviceSynchronize() { note("sync"); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { note("sync"); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)calloc(1, sizeof(long)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    std::lock_guard<std::mutex> g(mu);
    *(long*)e = clock_ms;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { note("sync"); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(*(long*)b - *(long*)a);
    return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) { memset(a, 0, sizeof *a); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 4; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = nullptr; return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
}
