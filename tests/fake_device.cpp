// A HIP runtime without a device, for tests of the host engine's bookkeeping: loaded with
// RTLD_GLOBAL before libfciqmc.so, its functions take the place of the runtime's. Device
// memory is host memory of a settable size, kernels do nothing except that
//   - k_finalize advances every system that takes part and writes the record the test set,
//   - k_extend asks for the places the test set,
//   - k_spawn counts a fault when a buffer it would write to is not as large as the
//     descriptors say.
#include <hip/hip_runtime_api.h>

#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../paper_1305_6981_amd/csrc/engine.h"

using namespace fq;

namespace {
std::map<char *, size_t> g_mem;               // device allocations
size_t g_capacity = (size_t)64 << 30, g_used = 0;
std::map<const void *, std::string> g_kernels;
struct Launch {
    std::string name;
    EngineArgs args;
};
bool g_capturing = false;
std::vector<Launch> g_captured;
struct Graph {
    std::vector<Launch> launches;
};
long g_graphs = 0, g_faults = 0, g_spawns = 0;
IterRecord g_next{};
unsigned long long g_extend = 0;

void *map_bytes(size_t n) {
    void *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    return p == MAP_FAILED ? nullptr : p;
}
// Whether [p, p + n) lies in one device allocation.
bool holds(const void *p, size_t n) {
    auto it = g_mem.upper_bound((char *)p);
    if (!p || it == g_mem.begin()) return false;
    --it;
    return (char *)p + n <= it->first + it->second;
}
bool takes_part(const EngineArgs &a, int s) {
    const SysDesc &d = a.desc[s];
    return d.active && a.status[s] == 0 && d.iter < d.stop_at;
}
void run(const Launch &l) {
    const EngineArgs &a = l.args;
    if (l.name.find("k_spawn") != std::string::npos) {
        ++g_spawns;
        for (int s = 0; s < a.max_sys; ++s) {
            if (!takes_part(a, s)) continue;
            const SysDesc &d = a.desc[s];
            const size_t rb = 16 * (size_t)d.det_words, b0 = (size_t)d.gchunk0 * BPC, nb = (size_t)d.nbuckets;
            if (!holds((char *)a.recs + (size_t)d.rec0 * rb, nb * (size_t)d.rec_r * rb) ||
                !holds(a.bhist + b0, nb * 4) || !holds(a.bprev + b0, nb * 4) ||
                !holds(a.bext + b0, nb * 8) || !holds(a.unlisted + b0, nb * 4) ||
                !holds(a.chunk_sys + d.gchunk0, (size_t)d.nchunks * 4) ||
                !holds(a.chunk_local + d.gchunk0, (size_t)d.nchunks * 4) ||
                (a.list_cap > 0 && !holds(a.tiles, (size_t)a.list_cap * NLIST * 16)))
                ++g_faults;
        }
    } else if (l.name.find("k_finalize") != std::string::npos) {
        for (int s = 0; s < a.max_sys; ++s) {
            if (!takes_part(a, s)) continue;
            IterRecord r = g_next;
            r.iter = ++a.desc[s].iter;
            a.rec[(int64_t)s * REC_CAP + r.iter % REC_CAP] = r;
        }
    }
}
}  // namespace

#define FAKE extern "C" __attribute__((visibility("default")))

// ---- the test's side
FAKE void fake_capacity(size_t bytes) { g_capacity = bytes; }
FAKE size_t fake_used() { return g_used; }
FAKE long fake_faults() { return g_faults; }
FAKE long fake_spawns() { return g_spawns; }
FAKE long fake_graphs() { return g_graphs; }
FAKE void fake_extend(unsigned long long places) { g_extend = places; }
FAKE void fake_iteration(long nw, long nd, long spawns, long used, long born, long rec_max) {
    g_next.nw = nw;
    g_next.nd = nd;
    g_next.spawns = spawns;
    g_next.used = used;
    g_next.born = born;
    g_next.rec_max = rec_max;
    g_next.c0 = 1;
}

// ---- the runtime's side
FAKE hipError_t hipMalloc(void **p, size_t n) {
    *p = nullptr;
    if (n > g_capacity || g_used > g_capacity - n) return hipErrorOutOfMemory;
    *p = map_bytes(n ? n : 1);
    if (!*p) return hipErrorOutOfMemory;
    g_mem[(char *)*p] = n ? n : 1;
    g_used += n ? n : 1;
    return hipSuccess;
}
FAKE hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    auto it = g_mem.find((char *)p);
    if (it == g_mem.end()) return hipErrorInvalidValue;
    munmap(p, it->second);
    g_used -= it->second;
    g_mem.erase(it);
    return hipSuccess;
}
FAKE hipError_t hipMemGetInfo(size_t *fr, size_t *tot) {
    *fr = g_used < g_capacity ? g_capacity - g_used : 0;
    *tot = g_capacity;
    return hipSuccess;
}
FAKE hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    *p = std::malloc(n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
FAKE hipError_t hipHostFree(void *p) {
    std::free(p);
    return hipSuccess;
}
FAKE hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned int) {
    *d = h;
    return hipSuccess;
}
FAKE hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    if (n) std::memcpy(d, s, n);
    return hipSuccess;
}
FAKE hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
    if (n) std::memset(d, v, n);
    return hipSuccess;
}
FAKE hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
FAKE hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {   // (by its current name)
    std::memset((void *)p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
FAKE hipError_t hipGetSymbolAddress(void **p, const void *s) {
    *p = (void *)s;
    return hipSuccess;
}
FAKE hipError_t hipGetLastError() { return hipSuccess; }
FAKE const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "error"; }
FAKE hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
    *s = (hipStream_t)&g_capturing;
    return hipSuccess;
}
FAKE hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
FAKE hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
FAKE hipError_t hipEventCreate(hipEvent_t *e) {
    *e = (hipEvent_t)&g_capturing;
    return hipSuccess;
}
FAKE hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
FAKE hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
FAKE hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
FAKE hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
FAKE hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    g_capturing = true;
    g_captured.clear();
    return hipSuccess;
}
FAKE hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    g_capturing = false;
    *g = (hipGraph_t) new Graph{g_captured};
    return hipSuccess;
}
FAKE hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
    *x = (hipGraphExec_t) new Graph(*(Graph *)g);
    ++g_graphs;
    return hipSuccess;
}
FAKE hipError_t hipGraphDestroy(hipGraph_t g) {
    delete (Graph *)g;
    return hipSuccess;
}
FAKE hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
    delete (Graph *)x;
    --g_graphs;
    return hipSuccess;
}
FAKE hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
    for (const Launch &l : ((Graph *)x)->launches) run(l);
    return hipSuccess;
}
FAKE hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t) {
    const std::string &name = g_kernels[f];
    if (name.find("k_extend") != std::string::npos) {
        **(unsigned long long **)args[7] += g_extend;
        return hipSuccess;
    }
    const bool iterates = name.find("k_spawn") != std::string::npos || name.find("k_finalize") != std::string::npos;
    if (!iterates) return hipSuccess;
    const Launch l{name, *(const EngineArgs *)args[0]};
    if (g_capturing)
        g_captured.push_back(l);
    else
        run(l);
    return hipSuccess;
}
FAKE hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
FAKE hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) {
    *g = *b = dim3(1);
    *m = 0;
    *s = nullptr;
    return hipSuccess;
}
FAKE void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
FAKE void __hipUnregisterFatBinary(void **) {}
FAKE void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned int, void *,
                                void *, void *, void *, int *) {
    g_kernels[host] = name;
}
FAKE void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
