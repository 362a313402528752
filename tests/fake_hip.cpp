// A stand-in for the HIP runtime on machines without a GPU.  Loaded with
// RTLD_GLOBAL ahead of libsv.so it takes the library's runtime calls: memory
// is host memory, kernels are not run, and what the host side asked for is
// kept in a log and checked against HIP's documented limits.  Streams and
// events carry the set of work items ordered before them, so that a buffer
// freed (or a call returned) while work is still outstanding shows.
//   fake_fail(api, n)   the n-th call of api from now on fails (0: none)
//   fake_fail_always    every call of api fails (on = 1) or none does
//   fake_log            one line per call, since fake_clear
//   fake_undone         work items launched and not known to be complete
//   fake_bad_frees      buffers freed while work was outstanding
//   fake_lds_limit      dynamic LDS that a kernel may be given
// Two kernels act on memory: k_upload copies, and k_reduce counts its ticket
// up and leaves it so when the call's copies fail afterwards (an interrupted
// reduction); a ticket that is not zero at its launch is logged.
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

namespace {

struct Stream {
    std::set<long> before;          // work items ordered before the stream's next one
    bool capturing = false;
    int captured = 0;
};
struct Event {
    std::set<long> before;
};
struct Graph {
    int launches = 0;
};

std::string g_log;
std::set<long> g_undone;
long g_next = 1, g_bad_frees = 0;
std::map<std::string, int> g_fail;
std::set<std::string> g_fail_always;
std::map<const void*, std::string> g_kernels;
std::map<const void*, int> g_lds;      // dynamic LDS a kernel may use (64 KiB unless set)
int g_lds_limit = 160 * 1024;          // ... and that the device has
std::map<const void*, size_t> g_vars;
std::map<const void*, void*> g_var_mem;
std::map<void*, size_t> g_alloc;
Stream g_null;
struct Config {
    dim3 grid, block;
    size_t shmem;
    hipStream_t stream;
} g_config;
hipError_t g_last = hipSuccess;

Stream* of(hipStream_t s) { return s ? (Stream*)s : &g_null; }

bool fails(const char* api)
{
    if (g_fail_always.count(api)) return true;
    auto it = g_fail.find(api);
    if (it == g_fail.end() || --it->second > 0) return false;
    g_fail.erase(it);
    return true;
}

void note(const std::string& line) { g_log += line + "\n"; }
std::string hex(const void* p)
{
    char b[32];
    snprintf(b, sizeof b, "%p", p);
    return b;
}

void work(Stream* s)
{
    if (s->capturing) {
        ++s->captured;
        return;
    }
    const long id = g_next++;
    g_undone.insert(id);
    s->before.insert(id);
}

void done(const std::set<long>& ids)
{
    for (long i : ids) g_undone.erase(i);
}

void* take(size_t n)
{
    if (n == 0) n = 1;
    void* p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) return nullptr;
    g_alloc[p] = n;
    return p;
}

void give(void* p)
{
    if (!p) return;
    if (!g_undone.empty()) {
        ++g_bad_frees;
        note("free " + hex(p) + " with work outstanding");
    }
    auto it = g_alloc.find(p);
    if (it == g_alloc.end()) return;
    munmap(p, it->second);
    g_alloc.erase(it);
}

hipError_t fail(hipError_t e) { return g_last = e; }

}  // namespace

extern "C" {

const char* fake_log() { return g_log.c_str(); }
void fake_clear() { g_log.clear(); }
long fake_undone() { return (long)g_undone.size(); }
long fake_bad_frees() { return g_bad_frees; }
void fake_lds_limit(int bytes) { g_lds_limit = bytes; }
void fake_fail(const char* api, int n)
{
    if (n > 0) g_fail[api] = n;
    else g_fail.erase(api);
}
void fake_fail_always(const char* api, int on)
{
    if (on) g_fail_always.insert(api);
    else g_fail_always.erase(api);
}

// ---- registration ------------------------------------------------------------
void** __hipRegisterFatBinary(const void*)
{
    static void* m = nullptr;
    return &m;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*,
                           int*)
{
    g_kernels[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int) { g_vars[var] = size; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream)
{
    g_config = {grid, block, shmem, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* stream)
{
    *grid = g_config.grid, *block = g_config.block, *shmem = g_config.shmem, *stream = g_config.stream;
    return hipSuccess;
}

// ---- kernels -----------------------------------------------------------------
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t shmem, hipStream_t st)
{
    const std::string& name = g_kernels[f];
    char line[160];
    snprintf(line, sizeof line, " grid %u %u %u block %u lds %zu stream %p", g.x, g.y, g.z, b.x, shmem, (void*)st);
    const uint64_t lim = 1ull << 32;
    // work items per dimension stay below 2^32, workgroups take at most 1024 lanes
    if (!g.x || !g.y || !g.z || (uint64_t)g.x * b.x >= lim || (uint64_t)g.y * b.y >= lim ||
        (uint64_t)g.z * b.z >= lim || b.x * b.y * b.z > 1024 ||
        shmem > (size_t)(g_lds.count(f) ? g_lds[f] : 64 * 1024)) {
        note("refused " + name + line);
        return fail(hipErrorInvalidConfiguration);
    }
    if (fails("hipLaunchKernel")) return fail(hipErrorUnknown);
    note("launch " + name + line);
    if (!of(st)->capturing) {
        if (name.find("k_upload") != std::string::npos)
            memcpy(*(void**)args[0], args[2], (size_t) * (int*)args[1] * 16);
        if (name.find("k_reduce") != std::string::npos) {
            unsigned* ticket = *(unsigned**)args[13];
            if (*(void**)args[14]) {
                if (*ticket) note("stale ticket");
                *ticket = g_fail.count("hipMemcpyAsync") ? 1 : 0;
            }
        }
    }
    work(of(st));
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int value)
{
    note("attribute " + g_kernels[f]);
    if (value > g_lds_limit) return fail(hipErrorInvalidValue);
    g_lds[f] = value;
    return hipSuccess;
}

// ---- memory ------------------------------------------------------------------
hipError_t hipMalloc(void** p, size_t n)
{
    if (fails("hipMalloc") || !(*p = take(n))) return fail(hipErrorOutOfMemory);
    return hipSuccess;
}
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return hipMalloc(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    if (fails("hipHostMalloc") || !(*p = take(n))) return fail(hipErrorOutOfMemory);
    return hipSuccess;
}
hipError_t hipFree(void* p) { give(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { give(p); return hipSuccess; }
hipError_t hipFreeAsync(void* p, hipStream_t)
{
    auto it = g_alloc.find(p);
    if (it != g_alloc.end()) munmap(p, it->second), g_alloc.erase(it);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* freeb, size_t* total)
{
    *freeb = *total = 288ull * 1000 * 1000 * 1000;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st)
{
    if (fails("hipMemcpyAsync")) return fail(hipErrorUnknown);
    char line[96];
    snprintf(line, sizeof line, "copy kind %d bytes %zu stream %p", (int)k, n, (void*)st);
    note(line);
    memmove(d, s, n);
    work(of(st));
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t hgt, hipMemcpyKind,
                            hipStream_t st)
{
    for (size_t i = 0; i < hgt; ++i) memmove((char*)d + i * dp, (const char*)s + i * sp, w);
    work(of(st));
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st)
{
    memset(d, v, n);
    work(of(st));
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* var)
{
    void*& m = g_var_mem[var];
    if (!m) m = take(g_vars[var]);
    *p = m;
    return hipSuccess;
}

// ---- streams, events, graphs ---------------------------------------------------
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    if (fails("hipStreamCreateWithFlags")) return fail(hipErrorOutOfMemory);
    *s = (hipStream_t) new Stream();
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { delete (Stream*)s; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s)
{
    note("sync stream " + hex((void*)s));
    done(of(s)->before);
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = 0; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    if (fails("hipStreamWaitEvent")) return fail(hipErrorUnknown);
    const Event* ev = (Event*)e;
    of(s)->before.insert(ev->before.begin(), ev->before.end());
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t) new Event(); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    if (fails("hipEventRecord")) return fail(hipErrorUnknown);
    ((Event*)e)->before = of(s)->before;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { done(((Event*)e)->before); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e)
{
    for (long i : ((Event*)e)->before)
        if (g_undone.count(i)) return hipErrorNotReady;
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    of(s)->capturing = true;
    of(s)->captured = 0;
    note("capture stream " + hex((void*)s));
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g)
{
    of(s)->capturing = false;
    *g = (hipGraph_t) new Graph{of(s)->captured};
    note("captured " + std::to_string(of(s)->captured));
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t)
{
    *x = (hipGraphExec_t) new Graph(*(Graph*)g);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s)
{
    if (fails("hipGraphLaunch")) return fail(hipErrorUnknown);
    note("graph stream " + hex((void*)s));
    work(of(s));
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (Graph*)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { delete (Graph*)x; return hipSuccess; }

// ---- the rest ------------------------------------------------------------------
hipError_t hipGetLastError()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }

}  // extern "C"
