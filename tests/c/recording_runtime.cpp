// A stand-in for the HIP runtime that records what the host library does, for tests without a GPU: loaded
// (RTLD_GLOBAL) before libfmb.so, its symbols take the place of libamdhip64's.  Device memory is host
// memory, kernels do not run; a launch keeps its name, grid, stream and, of the backward kernels, the work
// items its blocks take.  A buffer that a launch was given counts as in use until something waits for
// that launch's stream; a copy into it before that is counted as an overwrite.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "fmb_internal.h"

using namespace fmb;

namespace {
struct Alloc {
    size_t bytes;
    hipStream_t stream;
    bool used;
};
struct Launch {
    std::string name;
    unsigned grid[3];
    hipStream_t stream;
    std::vector<BwdItem> items;
};
std::map<uintptr_t, Alloc> allocs;
std::map<const void *, std::string> names;
std::vector<Launch> launches;
size_t in_use = 0, limit = SIZE_MAX;
long counts[5] = {0, 0, 0, 0, 0};  // allocations, copies, overwrites, calls a capture refuses, syncs
bool capturing = false;
hipError_t last_error = hipSuccess;
struct Config {
    dim3 g, b;
    size_t sh;
    hipStream_t st;
} config;

std::map<uintptr_t, Alloc>::iterator find(const void *p)
{
    auto it = allocs.upper_bound((uintptr_t)p);
    if (it == allocs.begin()) return allocs.end();
    --it;
    return (uintptr_t)p < it->first + it->second.bytes ? it : allocs.end();
}
void use(const void *p, hipStream_t st)
{
    auto it = find(p);
    if (it == allocs.end()) return;
    it->second.used = true;
    it->second.stream = st;
}
void wait(hipStream_t st, bool all)
{
    ++counts[4];
    for (auto &a : allocs)
        if (all || a.second.stream == st) a.second.used = false;
}
// arguments of the kernels that read the library's own buffers: P Params, O FwdOut, I BwdIn, p pointer, i int
struct Sig {
    const char *name, *args;
} const kSigs[] = {
    {"10fwd_kernel", "POpp"},      {"10bwd_kernel", "PIpppp"},   {"11bwdr_kernel", "PIpppp"}, {"11bwdt_kernel", "PIppppp"},
    {"14fin_one_kernel", "Pppp"},  {"11fin1_kernel", "ppppp"},   {"12fin1s_kernel", "ppppipp"}, {"11fin2_kernel", "Ppppp"},
    {"12statt_kernel", "Ppppp"},   {"15stat_fin_kernel", "Ppppp"}, {"11fwdc_kernel", "POp"}, {"11bwdc_kernel", "PIpppp"},
    {"12statc_kernel", "Pppppp"},
};
}  // namespace

extern "C" {

long rr_count(int what) { return counts[what]; }
void rr_set_limit(long bytes) { limit = bytes < 0 ? SIZE_MAX : (size_t)bytes; }
long rr_in_use() { return (long)in_use; }
void rr_set_capturing(int on) { capturing = on != 0; }
int rr_launches() { return (int)launches.size(); }
void rr_clear() { launches.clear(); }
const char *rr_name(int i) { return launches[i].name.c_str(); }
void rr_grid(int i, unsigned *out) { memcpy(out, launches[i].grid, sizeof launches[i].grid); }
// the items of launch i's blocks: (view, ray0, span, g0, gc, slots, poff, moff) each
int rr_items(int i, int *out, int cap)
{
    int n = 0;
    for (const auto &it : launches[i].items) {
        if (n >= cap) break;
        const int v[8] = {it.view, it.ray0, it.span, it.g0, it.gc, it.slots, it.poff, it.moff};
        memcpy(out + 8 * n++, v, sizeof v);
    }
    return (int)launches[i].items.size();
}

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    names[host] = device;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t st)
{
    config = {g, b, sh, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *st)
{
    *g = config.g;
    *b = config.b;
    *sh = config.sh;
    *st = config.st;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 g, dim3, void **args, size_t, hipStream_t st)
{
    Launch l{names[f], {g.x, g.y, g.z}, st, {}};
    if (g.y > 65535 || g.z > 65535 || g.x == 0 || g.y == 0) return last_error = hipErrorInvalidConfiguration;
    for (const auto &s : kSigs) {
        if (l.name.find(s.name) == std::string::npos) continue;
        for (int a = 0; s.args[a]; ++a) {
            if (s.args[a] == 'p') use(*(void **)args[a], st);
            if (s.args[a] == 'P') {
                const Params &p = *(const Params *)args[a];
                for (const void *q : {(const void *)p.views, (const void *)p.scenes, (const void *)p.eta}) use(q, st);
            }
        }
        if (s.args[1] == 'I') {
            const BwdItem *items = *(const BwdItem **)args[2];
            const int *order = *(const int **)args[3];
            for (unsigned b = 0; b < g.x; ++b) l.items.push_back(items[order ? order[b] : (int)b]);
        }
    }
    launches.push_back(l);
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n)
{
    if (capturing) return ++counts[3], hipErrorStreamCaptureUnsupported;
    if (n > limit || in_use > limit - n) return last_error = hipErrorOutOfMemory;
    void *mem = calloc(n, 1);
    if (!mem) return last_error = hipErrorOutOfMemory;
    ++counts[0];
    *p = mem;
    allocs[(uintptr_t)*p] = {n, nullptr, false};
    in_use += n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    wait(nullptr, true);  // freeing waits for the device
    --counts[4];
    auto it = allocs.find((uintptr_t)p);
    in_use -= it->second.bytes;
    allocs.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    ++counts[1];
    auto it = find(d);
    if (it != allocs.end() && it->second.used && it->second.stream != st) ++counts[2];
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k)
{
    if (capturing) return ++counts[3], hipErrorStreamCaptureUnsupported;
    return hipMemcpyAsync(d, s, n, k, nullptr);
}
hipError_t hipDeviceSynchronize()
{
    if (capturing) return ++counts[3], hipErrorStreamCaptureUnsupported;
    wait(nullptr, true);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st)
{
    wait(st, false);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    capturing = true;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    capturing = false;
    *g = (hipGraph_t)0x1;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *e = (hipGraphExec_t)0x2;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e)
{
    *e = (hipEvent_t)0x3;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "recorded error"; }
hipError_t hipGetLastError()
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static void *mem = calloc(64 << 20, 1);
    *p = mem;
    return hipSuccess;
}

}  // extern "C"
