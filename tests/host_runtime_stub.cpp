// Driver for the library's host runtime on a machine without a GPU (test
// infrastructure, host code only).
//
// It defines the HIP calls that liblbm355 makes: device memory is host memory
// with its extent on record, allocations can be made to fail, and a launch runs
// nothing but has its arguments checked: every buffer of totals that a kernel
// would write or read must be allocated and as long as the launch needs.
// Captured launches are kept and checked again at every replay.
//
//   host_runtime_stub CASE     prints "ok" and exits 0, or the first problems and 1
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "lb.h"
#include "lb_internal.h"

using namespace lbm;

static std::map<char *, size_t> g_live;  // device allocations
// kernels by their host stubs (registered before this file's globals exist)
static std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> fn;
    return fn;
}
static int g_allow = -1;                 // allocations before the first failing one (-1: all work)
static int g_launches = 0, g_problems = 0;

static void problem(const std::string &what)
{
    if (++g_problems <= 8) std::printf("PROBLEM %s\n", what.c_str());
}

static void expect(bool ok, const char *what)
{
    if (!ok) problem(std::string(what) + " (last error: " + lb_last_error() + ")");
}

static void need(const void *p, size_t bytes, const std::string &what)
{
    char *c = static_cast<char *>(const_cast<void *>(p));
    auto it = g_live.upper_bound(c);
    if (c && it != g_live.begin()) {
        --it;
        if (c >= it->first && c + bytes <= it->first + it->second) return;
    }
    problem(what + (c ? ": not allocated, or too short" : ": null"));
}

static void check_totals(const TotalsArgs &t, int steps, const std::string &name)
{
    need(t.partials, (size_t)t.nparts * t.nc * sizeof(double), name + ": partials");
    need(t.gpartials, (size_t)(t.nparts + kRedChunk - 1) / kRedChunk * t.nc * steps * sizeof(double), name + ": chunk sums");
    need(t.ring, (size_t)kRingCap * 4 * sizeof(double), name + ": ring");
    need(t.step_counter, sizeof(unsigned long long), name + ": step counter");
}

struct Launch {
    std::string name;
    std::vector<char> args;
    int nsteps;
};

static void check_launch(const Launch &l)
{
    ++g_launches;
    if (l.name.find("reduce_totals") != std::string::npos) {
        const TotalsArgs *t = reinterpret_cast<const TotalsArgs *>(l.args.data());
        for (int k = 0; k < l.nsteps; ++k) check_totals(t[k], l.nsteps, l.name);
    } else if (!l.args.empty()) {
        const StepArgs &a = *reinterpret_cast<const StepArgs *>(l.args.data());
        const size_t nc = a.split.m1 != 0.0 && !a.fx_field ? 8 : 4;
        const size_t tiles = ((size_t)a.nslots + kBlock - 1) / kBlock;
        need(a.partials, tiles * nc * sizeof(double), l.name + ": own partials");
        for (int k = 0; k < a.nprev; ++k) check_totals(a.prev[k], a.nprev, l.name);
    }
}

static bool g_capturing = false;
static std::vector<Launch> g_captured;
static dim3 g_grid, g_block;

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, dim3 *, dim3 *, int *)
{
    kernels()[host] = device;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) { g_grid = g; g_block = b; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s)
{
    *g = g_grid; *b = g_block; *m = 0; *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3, dim3, void **args, size_t, hipStream_t)
{
    Launch l{kernels()[fn], {}, 0};
    size_t bytes = 0;
    if (l.name.find("reduce_totals") != std::string::npos) {
        bytes = kMaxSteps * sizeof(TotalsArgs);
        l.nsteps = *static_cast<int *>(args[1]);
    } else if (l.name.find("step_vec") != std::string::npos || l.name.find("step_site") != std::string::npos) {
        bytes = sizeof(StepArgs);
    }
    if (bytes) l.args.assign(static_cast<char *>(args[0]), static_cast<char *>(args[0]) + bytes);
    if (g_capturing) g_captured.push_back(l);
    else check_launch(l);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    if (g_allow == 0) return hipErrorOutOfMemory;
    if (g_allow > 0) --g_allow;
    *p = std::calloc(n ? n : 1, 1);
    g_live[static_cast<char *>(*p)] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (p && !g_live.erase(static_cast<char *>(p))) problem("hipFree of memory that is not allocated");
    return hipSuccess;  // kept mapped: an address is not given out twice
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) { *p = {}; p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) { *a = {}; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 4; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static char *m = static_cast<char *>(std::calloc((size_t)32 << 20, 1));
    g_live[m] = (size_t)32 << 20;
    *p = m;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = reinterpret_cast<hipStream_t>(2); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { g_capturing = true; g_captured.clear(); return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    g_capturing = false;
    *g = reinterpret_cast<hipGraph_t>(new std::vector<Launch>(g_captured));
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    *e = reinterpret_cast<hipGraphExec_t>(new std::vector<Launch>(*reinterpret_cast<std::vector<Launch> *>(g)));
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete reinterpret_cast<std::vector<Launch> *>(g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { delete reinterpret_cast<std::vector<Launch> *>(e); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t)
{
    for (const Launch &l : *reinterpret_cast<std::vector<Launch> *>(e)) check_launch(l);
    return hipSuccess;
}
}

static lb_lattice *make(int nx, int ny, int nz, int storage, bool solids)
{
    std::vector<uint8_t> flags((size_t)nx * ny * nz, 0);
    if (solids) flags[1] = 1;
    lb_lattice *h = lb_create_ex(nx, ny, nz, 0.7, solids ? flags.data() : nullptr, storage, nullptr);
    if (!h) {
        std::printf("PROBLEM creation: %s\n", lb_last_error());
        std::exit(1);
    }
    return h;
}

// The tuner's totals ring holds every step of the longest sweep.
static void tuner_ring()
{
    lb_lattice *h = make(64, 16, 16, LB_F16S, true);
    expect(lb_tune(h, 1000) == LB_OK, "tune");
    expect(lb_step(h, 3) == LB_OK, "step");
    lb_destroy(h);
}

// Setting or clearing a force field changes the step kernel's width, and with
// it the number of partials: when memory runs out in between, the lattice
// steps on with buffers that exist.
static void force_field_memory()
{
    lb_lattice *h = make(32, 16, 12, LB_F32, true);
    void *fx = nullptr;
    (void)hipMalloc(&fx, 32 * 16 * 12 * sizeof(float));
    expect(lb_step(h, 70) == LB_OK, "step");
    g_allow = 1;  // the field itself
    (void)lb_set_force_field(h, static_cast<float *>(fx));
    expect(lb_step(h, 70) == LB_OK && lb_step(h, 1) == LB_OK, "step with the field");
    g_allow = 0;
    expect(lb_set_force_field(h, nullptr) == LB_OK, "clearing the field needs no memory");
    expect(lb_step(h, 70) == LB_OK && lb_step(h, 1) == LB_OK, "step without the field");
    lb_destroy(h);
}

// A sweep that finds no memory for its widest grid leaves the lattice, and its
// captured runs, as they were.
static void tuner_memory()
{
    lb_lattice *h = make(128, 256, 256, LB_F32, true);
    expect(lb_step(h, 64) == LB_OK, "step");
    for (int allow = 0; allow < 4; ++allow) {
        g_allow = allow;
        (void)lb_tune(h, 2);
        g_allow = -1;
        expect(lb_step(h, 64) == LB_OK && lb_step(h, 1) == LB_OK, "step after a failed sweep");
    }
    lb_destroy(h);
}

int main(int argc, char **argv)
{
    const std::string which = argc > 1 ? argv[1] : "";
    if (which == "tuner_ring") tuner_ring();
    else if (which == "force_field_memory") force_field_memory();
    else if (which == "tuner_memory") tuner_memory();
    else {
        std::printf("unknown case %s\n", which.c_str());
        return 2;
    }
    if (g_launches == 0) problem("no launch was seen");
    if (g_problems) return 1;
    std::printf("ok %d launches\n", g_launches);
    return 0;
}
