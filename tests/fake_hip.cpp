// A HIP runtime without a GPU, for tests of the library's host code. Loaded
// with global visibility before liblbm.so, its functions take the place of the
// runtime's: device memory is lazily mapped host memory counted against a
// limit, kernels are not run but logged by name, asynchronous copies into
// pinned memory happen when their stream or event is waited for, and calls
// can be made to fail. Two devices. What the tests read is at the end.
#include <hip/hip_runtime_api.h>

#include <cxxabi.h>
#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {

constexpr int kDevices = 2;

struct Block {
    size_t bytes;
    int device;  // -1: pinned host memory
};
struct FakePool {
    int device;
    size_t keep = 0;
    std::multimap<size_t, char*> idle;
};
struct Copy {
    void* dst;
    const void* src;
    size_t bytes;
};
struct FakeStream {
    int device;
    std::deque<Copy> copies;
};
struct FakeEvent {
    int device;
    FakeStream* stream = nullptr;
    size_t at = 0;  // log length when it was recorded
};

std::recursive_mutex g_mu;
using Hold = std::lock_guard<std::recursive_mutex>;
thread_local int t_device = 0;
size_t g_limit[kDevices] = {size_t(288) << 30, size_t(288) << 30};
size_t g_used[kDevices] = {};
std::map<char*, Block> g_blocks;
std::map<char*, FakePool*> g_pooled;  // blocks handed out by a pool (null: the device's default)
std::map<const void*, std::string> g_kernels;
std::vector<std::string> g_log;
std::string g_text, g_fast;
std::map<std::string, std::pair<int, int>> g_fail;  // function: calls until it fails, error
FakeStream g_null[kDevices] = {{0, {}}, {1, {}}};

FakeStream* of(hipStream_t s) { return s ? (FakeStream*)s : &g_null[t_device]; }
void say(const std::string& s) { g_log.push_back(s); }
void drain(FakeStream* s)
{
    for (const Copy& c : s->copies) std::memcpy(c.dst, c.src, c.bytes);
    s->copies.clear();
}
int failing(const char* fn)
{
    auto it = g_fail.find(fn);
    if (it == g_fail.end() || it->second.first-- != 0) return 0;
    const int e = it->second.second;
    g_fail.erase(it);
    return e;
}
#define FAKE(fn)                                                \
    Hold hold(g_mu);                                            \
    if (const int fail_ = failing(fn)) return (hipError_t)fail_

char* map_bytes(size_t n, int device)
{
    void* p = mmap(nullptr, n ? n : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) std::abort();
    g_blocks[(char*)p] = {n, device};
    return (char*)p;
}
char* take(size_t n, int device)
{
    if (g_used[device] + n > g_limit[device]) return nullptr;
    g_used[device] += n;
    return map_bytes(n, device);
}
void give(char* p)
{
    const auto it = g_blocks.find(p);
    if (it == g_blocks.end()) std::abort();  // not ours, or freed twice
    if (it->second.device >= 0) g_used[it->second.device] -= it->second.bytes;
    munmap(p, it->second.bytes ? it->second.bytes : 1);
    g_blocks.erase(it);
}
const Block* find(const void* p)
{
    auto it = g_blocks.upper_bound((char*)p);
    if (it == g_blocks.begin()) return nullptr;
    --it;
    return (char*)p < it->first + it->second.bytes ? &it->second : nullptr;
}

}  // namespace

extern "C" {

// registration and launches
void** __hipRegisterFatBinary(const void*)
{
    static void* h;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    Hold hold(g_mu);
    int st = 0;
    std::string s = name;
    for (size_t i; (i = s.find("DF16_")) != std::string::npos;) s.replace(i, 5, "Dh");  // _Float16, as the demangler knows it
    char* d = abi::__cxa_demangle(s.c_str(), nullptr, nullptr, &st);
    if (d) s = d;
    std::free(d);
    if (s.rfind("void ", 0) == 0) s = s.substr(5);
    size_t i = 0;
    for (int depth = 0; i < s.size() && (depth || s[i] != '('); ++i) depth += s[i] == '<' ? 1 : (s[i] == '>' ? -1 : 0);
    g_kernels[host] = s.substr(0, i);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
static thread_local struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t st;
} t_cfg;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st)
{
    t_cfg = {g, b, lds, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st)
{
    *g = t_cfg.grid;
    *b = t_cfg.block;
    *lds = t_cfg.lds;
    *st = t_cfg.st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t)
{
    FAKE("hipLaunchKernel");
    say("launch " + g_kernels[f]);
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }

// devices
hipError_t hipGetDevice(int* d)
{
    *d = t_device;
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    if (d < 0 || d >= kDevices) return hipErrorInvalidDevice;
    t_device = d;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void)
{
    Hold hold(g_mu);
    drain(&g_null[t_device]);
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950:sramecc+");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t)
{
    *n = 2;
    return hipSuccess;
}

// memory
hipError_t hipMalloc(void** p, size_t n)
{
    FAKE("hipMalloc");
    *p = take(n, t_device);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p)
{
    Hold hold(g_mu);
    if (p) give((char*)p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    FAKE("hipHostMalloc");
    *p = map_bytes(n, -1);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    Hold hold(g_mu);
    if (p) give((char*)p);
    return hipSuccess;
}
hipError_t hipMemPoolCreate(hipMemPool_t* m, const hipMemPoolProps* props)
{
    FAKE("hipMemPoolCreate");
    *m = (hipMemPool_t) new FakePool{props->location.id, 0, {}};
    return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t m, hipMemPoolAttr a, void* v)
{
    if (a == hipMemPoolAttrReleaseThreshold) ((FakePool*)m)->keep = (size_t)*(uint64_t*)v;
    return hipSuccess;
}
hipError_t hipMemPoolTrimTo(hipMemPool_t m, size_t keep)
{
    Hold hold(g_mu);
    FakePool* p = (FakePool*)m;
    size_t held = 0;
    for (auto& k : p->idle) held += k.first;
    while (held > keep && !p->idle.empty()) {
        held -= p->idle.begin()->first;
        give(p->idle.begin()->second);
        p->idle.erase(p->idle.begin());
    }
    return hipSuccess;
}
hipError_t hipMemPoolDestroy(hipMemPool_t m)
{
    hipMemPoolTrimTo(m, 0);
    delete (FakePool*)m;
    return hipSuccess;
}
hipError_t hipMallocFromPoolAsync(void** out, size_t n, hipMemPool_t m, hipStream_t st)
{
    FAKE("hipMallocFromPoolAsync");
    FakePool* p = (FakePool*)m;
    if (p->device != of(st)->device) say("foreign scratch");
    auto it = p->idle.lower_bound(n);
    char* q;
    if (it != p->idle.end()) {
        q = it->second;
        p->idle.erase(it);
    } else {
        q = take(n, p->device);
    }
    if (q) g_pooled[q] = p;
    *out = q;
    return q ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipMallocAsync(void** out, size_t n, hipStream_t st)
{
    FAKE("hipMallocAsync");
    char* q = take(n, of(st)->device);
    if (q) g_pooled[q] = nullptr;
    *out = q;
    return q ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFreeAsync(void* v, hipStream_t)
{
    Hold hold(g_mu);
    char* q = (char*)v;
    FakePool* p = g_pooled.at(q);
    g_pooled.erase(q);
    if (!p) {
        give(q);
        return hipSuccess;
    }
    size_t held = g_blocks[q].bytes;
    for (auto& k : p->idle) held += k.first;
    p->idle.emplace(g_blocks[q].bytes, q);
    if (held > p->keep) hipMemPoolTrimTo((hipMemPool_t)p, p->keep);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p)
{
    Hold hold(g_mu);
    const Block* b = find(p);
    if (!b) return hipErrorInvalidValue;
    a->type = b->device < 0 ? hipMemoryTypeHost : hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    static char* scratch;
    Hold hold(g_mu);
    if (!scratch) scratch = map_bytes(size_t(64) << 20, -1);
    *p = scratch;
    return hipSuccess;
}
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t)
{
    FAKE("hipMemsetAsync");
    return hipSuccess;  // all memory is fresh and zero
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t st)
{
    FAKE("hipMemcpyAsync");
    const Block* b = find(dst);
    if (b && b->device < 0) of(st)->copies.push_back({dst, src, n});
    else std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind)
{
    Hold hold(g_mu);
    std::memcpy(dst, src, n);
    return hipSuccess;
}

// streams, events, graphs
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = (hipStream_t) new FakeStream{t_device, {}};
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    delete (FakeStream*)s;
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d)
{
    *d = of(s)->device;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    FAKE("hipStreamSynchronize");
    drain(of(s));
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    FAKE("hipEventCreateWithFlags");
    *e = (hipEvent_t) new FakeEvent{t_device, nullptr, 0};
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete (FakeEvent*)e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    FAKE("hipEventRecord");
    if (((FakeEvent*)e)->device != of(s)->device) return hipErrorInvalidHandle;  // as the runtime does
    ((FakeEvent*)e)->stream = of(s);
    ((FakeEvent*)e)->at = g_log.size();
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    FAKE("hipEventSynchronize");
    if (((FakeEvent*)e)->stream) drain(((FakeEvent*)e)->stream);
    return hipSuccess;
}
// 0.01 ms if a kernel whose name holds the text of fake_fast ran between, else 1
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    Hold hold(g_mu);
    *ms = 1.0f;
    for (size_t k = ((FakeEvent*)a)->at; k < ((FakeEvent*)b)->at; ++k)
        if (!g_fast.empty() && g_log[k].find(g_fast) != std::string::npos) *ms = 0.01f;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    *g = (hipGraph_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    *x = (hipGraphExec_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    std::free((void*)g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    std::free((void*)x);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t)
{
    FAKE("hipGraphLaunch");
    say("graph");
    return hipSuccess;
}

// for the tests
const char* fake_log(void)  // and clear it
{
    Hold hold(g_mu);
    g_text.clear();
    for (const std::string& s : g_log) g_text += s + "\n";
    g_log.clear();
    return g_text.c_str();
}
void fake_fail(const char* fn, int after, int error)  // the call after the next `after` ones, once
{
    Hold hold(g_mu);
    g_fail[fn] = {after, error};
}
void fake_limit(int device, size_t bytes)
{
    Hold hold(g_mu);
    g_limit[device] = bytes;
}
size_t fake_used(int device)
{
    Hold hold(g_mu);
    return g_used[device];
}
int fake_pending(void* stream)  // copies not yet waited for
{
    Hold hold(g_mu);
    return (int)of((hipStream_t)stream)->copies.size();
}
void fake_fast(const char* text)
{
    Hold hold(g_mu);
    g_fast = text;
}

}  // extern "C"
