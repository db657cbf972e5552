// A stand-in for the HIP runtime on the CPU (preloaded by test_host_objects.py):
// device memory is host memory, kernels do nothing, and streams, events and
// captured graphs are counted, with what each graph was captured through.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

namespace {

struct Captured {
    std::set<void *> through;      // streams and events
};
std::set<void *> streams, events;
std::map<void *, Captured> graphs, execs;
bool capturing = false;
Captured capture;
std::set<void *> recorded;         // events recorded in the capture in progress
std::map<const void *, std::string> names;   // kernels by their host stubs
std::map<std::string, long> launched;
std::string fails;                 // the next call of this name fails
int misuses = 0;
long limit = 0;                    // the most bytes of one allocation (0: any)
long launches = 0, bad_grids = 0, waits = 0;

bool failing(const char *what)
{
    if (fails != what) return false;
    fails.clear();
    return true;
}
template <typename H>
hipError_t make(std::set<void *> &in, H *out)
{
    *out = (H)malloc(8);
    in.insert((void *)*out);
    return hipSuccess;
}
hipError_t drop(std::set<void *> &from, void *what)
{
    for (auto &e : execs)
        if (e.second.through.count(what)) ++misuses;   // a graph that is still there was captured through it
    if (!from.erase(what)) ++misuses;
    free(what);
    return hipSuccess;
}

}  // namespace

extern "C" {
void stub_limit(long bytes) { limit = bytes; }
void stub_fail(const char *what) { fails = what; }
int stub_misuses() { return misuses; }
int stub_live() { return (int)(streams.size() + events.size() + graphs.size() + execs.size()); }
long stub_waits() { return waits; }
long stub_launches() { return launches; }
// launches of the kernels whose (mangled) names hold `part`, since the last call
long stub_launched(const char *part)
{
    long n = 0;
    for (auto &l : launched)
        if (l.first.find(part) != std::string::npos) n += l.second;
    return n;
}
void stub_forget() { launched.clear(); }
long stub_bad_grids() { return bad_grids; }

hipError_t hipMalloc(void **p, size_t n)
{
    *p = limit && (long)n > limit ? nullptr : malloc(n + 256);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { if (capturing) ++misuses; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return make(streams, s); }
hipError_t hipStreamDestroy(hipStream_t s) { return drop(streams, s); }
hipError_t hipEventCreate(hipEvent_t *e) { return make(events, e); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return make(events, e); }
hipError_t hipEventDestroy(hipEvent_t e) { return drop(events, e); }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 1; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    if (failing("hipEventRecord")) return hipErrorUnknown;
    if (capturing && capture.through.count(s)) {
        capture.through.insert(e);
        recorded.insert(e);
    }
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    if (failing("hipStreamWaitEvent")) return hipErrorUnknown;
    ++waits;
    if (capturing && recorded.count(e)) capture.through.insert(s);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st)
{
    *st = capturing && capture.through.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    if (capturing) ++misuses;
    if (failing("hipStreamBeginCapture")) return hipErrorUnknown;
    capturing = true;
    capture = Captured();
    capture.through.insert(s);
    recorded.clear();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    capturing = false;
    *g = nullptr;
    if (failing("hipStreamEndCapture")) return hipErrorUnknown;
    *g = (hipGraph_t)malloc(8);
    graphs[*g] = capture;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { graphs.erase(g); free(g); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    if (failing("hipGraphInstantiate")) return hipErrorUnknown;
    *e = (hipGraphExec_t)malloc(8);
    execs[*e] = graphs[g];
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { execs.erase(e); free(e); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return failing("hipGraphLaunch") ? hipErrorUnknown : hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static char *static_ws = (char *)aligned_alloc(256, 16 << 20);
    *p = static_ws;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return failing("hipGetLastError") ? hipErrorUnknown : hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipLaunchKernel(const void *host, dim3 g, dim3 b, void **, size_t, hipStream_t)
{
    ++launches;
    ++launched[names[host]];
    if (g.x == 0 || g.y == 0 || g.z == 0 || (unsigned long)g.x * b.x > 0xFFFFFFFFul) ++bad_grids;
    return hipSuccess;
}
static thread_local dim3 grid, block;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) { grid = g; block = b; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *n, hipStream_t *s)
{
    *g = grid;
    *b = block;
    *n = 0;
    *s = nullptr;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}
