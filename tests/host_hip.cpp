// A HIP runtime and kernel launchers that do nothing, for host tests of dsve_api.cpp: device memory is host
// memory, kernels are counted, and what a test sets by name (fake_set) the calls below report.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

#include "dsve_internal.hpp"

using namespace dsve;

static std::map<std::string, long> V;
static std::set<const void *> live;
static hipError_t last = hipSuccess;   // as the runtime keeps it: until it is asked for
static double clock_ms = 0.0;

static hipError_t give(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}
static hipError_t launched(const char *what, float ms = 0.f)
{
    ++V[what];
    clock_ms += ms;
    return hipGetLastError();
}

extern "C" {

void fake_reset()
{
    V.clear();
    clock_ms = 0.0;
    last = hipSuccess;
    V["cus"] = V["mask"] = 256;   // compute units, and those the stream may use
    V["per_cu"] = 1;              // workgroups of k_parts on each
    V["us_parts"] = V["us_step"] = 1;
}
void fake_set(const char *name, long v) { V[name] = v; }
long fake_get(const char *name) { return V[name]; }
int fake_live(long p) { return (int)live.count((const void *)p); }

hipError_t hipGetLastError(void)
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int)
{
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = (int)V["cus"];
    std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)8; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipExtStreamGetCUMask(hipStream_t, uint32_t n, uint32_t *m)
{
    if (V["mask_error"]) return give(hipErrorInvalidValue);
    for (uint32_t k = 0; k < 32 * n; ++k)
        if ((long)k < V["mask"]) m[k / 32] |= 1u << (k % 32);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = V["capturing"] ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::calloc(1, n ? n : 1);
    live.insert(*p);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    V["freed"] = (long)p;
    live.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t) new double(0.0); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete (double *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { *(double *)e = clock_ms; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(*(double *)b - *(double *)a);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { V["recording"] = 1; V["recorded"] = 0; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { V["recording"] = 0; *g = (hipGraph_t)8; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    ++V["captures"];
    *e = (hipGraphExec_t) new long(V["recorded"]);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { delete (long *)e; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t)
{
    clock_ms += 1e-3f * (float)V["us_step"] * (float)*(long *)e;
    ++V["graphs"];
    return hipSuccess;
}

}  // extern "C"

namespace dsve {

hipError_t launch_step(const StepArgs &a, int, int, int, int, int, hipStream_t)
{
    V["table"] = a.segments ? (long)a.segments : (long)a.tile_chan;
    V["look"] = a.amax_check;
    if (V["recording"]) {
        ++V["recorded"];
        return hipSuccess;
    }
    return launched("steps", 1e-3f * (float)V["us_step"]);
}
int packed_blocks_per_cu(int, int, int, int, int64_t) { return 4; }
hipError_t launch_cfl(const CflArgs &, int, int, hipStream_t) { return launched("cfl"); }
hipError_t launch_fluct(const FluctArgs &, int, int, int, hipStream_t) { return launched("fluct"); }
hipError_t launch_cell_update(const double *, const double *, const double *, const ChanInfo *, double, int64_t,
                              double *, double *, double *, hipStream_t)
{
    return launched("update");
}
hipError_t launch_start(const StepArgs &, int, int, bool, hipStream_t) { return launched("start"); }
hipError_t launch_cfl_one(const CflOneArgs &, int, int, hipStream_t) { return launched("cfl_one"); }
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t)
{
    for (int64_t i = 0; i < n; ++i) p[i] = v;
    return launched("fill");
}
hipError_t launch_fill_u32(unsigned int *p, int64_t n, unsigned int v, hipStream_t)
{
    for (int64_t i = 0; i < n; ++i) p[i] = v;
    return launched("fill");
}
hipError_t launch_resident(const ResidentArgs &a, int, int, int, int, int, hipStream_t)
{
    return launched("resident", 1e-3f * (float)V["us_parts"] * (float)a.n_steps);
}
int parts_per_cu(int, int, int) { return (int)V["per_cu"]; }
hipError_t launch_parts(const PartArgs &a, int, int, int, int, hipStream_t)
{
    a.flags[0] |= (unsigned)V["raise"];
    V["wait"] = (long)a.wait_ticks;
    V["hold"] = a.hold_part;
    return launched("parts", 1e-3f * (float)V["us_parts"] * (float)a.n_steps);
}
int amax_split_of_kernels() { return kAmaxSplitMax; }
hipError_t launch_copy_u64(unsigned long long *d, const unsigned long long *s, int64_t n, hipStream_t)
{
    std::memcpy(d, s, sizeof *d * (size_t)n);
    return launched("copy");
}
hipError_t noalloc_scratch(int, void **p)
{
    static char *scratch = nullptr;
    *p = nullptr;
    if (V["scratch_error"]) return give(hipErrorInvalidSymbol);
    if (!scratch) scratch = (char *)std::calloc(1, kNoAllocScratchBytes);
    *p = scratch;
    return hipSuccess;
}

}  // namespace dsve
