// host_device.hip -- a stand-in for the GPU in host memory, linked with the host side of the library (api.hip compiled
// for the host alone) by test_host_lists.py.  Allocations are counted and can be made to fail; a step "launch" computes
// nothing: it checks that every list, item and array it was given lies in a live allocation, adds a modelled time, and
// a residual reduction writes the sums that the test asked for.  A captured graph is the list of its launches, checked
// again at each replay.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "ifdlbm_internal.h"

namespace {

std::map<const char*, size_t> live;       // device allocations
size_t live_bytes = 0, peak_bytes = 0;
long allocations_left = -1, pinned_left = -1;   // until an allocation fails (-1: never)
hipError_t last_error = hipSuccess;       // as a launch reports it
int faults = 0;
std::string first_fault, last_kernel;
std::vector<int> converged;               // per cavity: what the next residual reduction reports
double clock_ms = 0.0;
int cheap_rows = 0;                       // item rows at which the modelled march is fastest
bool capturing = false;
std::vector<std::function<void()>> recorded;

void fault(const std::string& what)
{
    if (!faults++) first_fault = what;
}

bool inside(const void* p, size_t bytes)
{
    const char* c = static_cast<const char*>(p);
    auto it = live.upper_bound(c);
    if (!p || it == live.begin()) return false;
    --it;
    return c >= it->first && c + bytes <= it->first + it->second;
}

void check(const void* p, size_t bytes, const char* what)
{
    if (bytes && !inside(p, bytes)) fault(what);
}

void submit(std::function<void()> f)
{
    if (capturing)
        recorded.push_back(std::move(f));
    else
        f();
}

hipError_t take(void** p, size_t bytes, long& left)
{
    if (left == 0) return last_error = hipErrorOutOfMemory;
    if (left > 0) --left;
    *p = std::malloc(bytes);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}

hipError_t step(const char* kernel, int prec, const ifd::StepArgs& a, const ifd::StripItem* items, int w0, int nw, bool residual)
{
    const std::string name = kernel;
    submit([=] {
        last_kernel = name;
        const size_t fs = prec == ifd::P_FP64 ? 8 : prec == ifd::P_FP16DEV ? 2 : 4, ls = prec == ifd::P_FP64 ? 8 : 4;
        if (!inside(items + w0, (size_t)nw * sizeof(ifd::StripItem))) return fault("item list");
        int rows = 0;
        for (int w = w0; w < w0 + nw; ++w) {
            const ifd::StripItem& it = items[w];
            if (it.unit < 0) continue;
            if (!inside(a.desc + it.cav, sizeof(ifd::CavityDesc))) return fault("descriptor");
            const ifd::CavityDesc& c = a.desc[it.cav];
            if (it.i0 < 0 || it.i0 >= it.i1 || it.i1 > c.nx || it.j0 < 0 || it.j0 >= it.j1 || it.j1 > c.ny) return fault("item");
            rows = it.j1 - it.j0 > rows ? it.j1 - it.j0 : rows;
            check(static_cast<const char*>(a.f_in) + c.f_off * fs, 9 * c.plane * fs, "f in");
            check(static_cast<const char*>(a.f_out) + c.f_off * fs, 9 * c.plane * fs, "f out");
            check(static_cast<const char*>(a.l_in) + c.l_off * ls, c.plane * ls, "lambda in");
            check(static_cast<const char*>(a.l_out) + c.l_off * ls, c.plane * ls, "lambda out");
            if (residual) check(a.partial + (int64_t)it.unit * ifd::kPartials, ifd::kPartials * sizeof(double), "partial sums");
        }
        clock_ms += name == "tile" ? 1.0 : 10.0 + 0.1 * std::abs(rows - cheap_rows);
    });
    return hipGetLastError();
}

}  // namespace

extern "C" {
// ------------------------------------------------------------ for the test
void host_reset(long fail_after, long pinned_after)
{
    allocations_left = fail_after;
    pinned_left = pinned_after;
    faults = 0;
    first_fault.clear();
    last_error = hipSuccess;
    peak_bytes = live_bytes;
}
void host_converge(const int* flags, int n) { converged.assign(flags, flags + n); }
void host_cheap_rows(int rows) { cheap_rows = rows; }
int host_faults(char* text, int size)
{
    std::snprintf(text, size, "%s", first_fault.c_str());
    return faults;
}
void host_last_kernel(char* text, int size) { std::snprintf(text, size, "%s", last_kernel.c_str()); }
long host_peak_bytes() { return (long)peak_bytes; }
long host_live_bytes() { return (long)live_bytes; }

// ----------------------------------------------------------- the runtime
hipError_t hipMalloc(void** p, size_t bytes)
{
    const hipError_t e = take(p, bytes, allocations_left);
    if (e != hipSuccess) return e;
    live[static_cast<char*>(*p)] = bytes;
    live_bytes += bytes;
    peak_bytes = live_bytes > peak_bytes ? live_bytes : peak_bytes;
    return e;
}
hipError_t hipFree(void* p)
{
    if (!p) return hipSuccess;
    auto it = live.find(static_cast<char*>(p));
    if (it == live.end()) {
        fault("free of no allocation");
        return hipErrorInvalidValue;
    }
    live_bytes -= it->second;
    live.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { return take(p, bytes, pinned_left); }
hipError_t hipHostFree(void* p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind kind, hipStream_t)
{
    const bool to = kind != hipMemcpyDeviceToHost, from = kind != hipMemcpyHostToDevice;
    if ((to && !inside(dst, bytes)) || (from && !inside(src, bytes))) {
        fault("copy");
        return hipErrorInvalidValue;
    }
    if (!(to && from)) std::memcpy(dst, src, bytes);   // the states copied between device arrays hold nothing
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t bytes, hipStream_t)
{
    if (!inside(p, bytes)) {
        fault("memset");
        return hipErrorInvalidValue;
    }
    std::memset(p, v, bytes);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = reinterpret_cast<hipStream_t>(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    capturing = true;
    recorded.clear();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    capturing = false;
    *g = reinterpret_cast<hipGraph_t>(new std::vector<std::function<void()>>(recorded));
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t)
{
    *x = reinterpret_cast<hipGraphExec_t>(new std::vector<std::function<void()>>(*reinterpret_cast<std::vector<std::function<void()>>*>(g)));
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete reinterpret_cast<std::vector<std::function<void()>>*>(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    delete reinterpret_cast<std::vector<std::function<void()>>*>(x);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t)
{
    for (auto& f : *reinterpret_cast<std::vector<std::function<void()>>*>(x)) f();
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = reinterpret_cast<hipEvent_t>(new double(0.0));
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete reinterpret_cast<double*>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    *reinterpret_cast<double*>(e) = clock_ms;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(*reinterpret_cast<double*>(b) - *reinterpret_cast<double*>(a));
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }

}  // extern "C"

// ------------------------------------------------------------ the launches
namespace ifd {

hipError_t launch_seed_bump(uint32_t* ctr, hipStream_t)
{
    submit([=] { check(ctr, sizeof(uint32_t), "seed"); });
    return hipSuccess;
}
hipError_t launch_staged_step(int, const StepArgs& a, const NodeBlock* blocks, int b0, int nb, bool residual, hipStream_t)
{
    submit([=] {
        last_kernel = "staged";
        check(blocks + b0, (size_t)nb * sizeof(NodeBlock), "block list");
        if (residual) check(a.partial + (int64_t)b0 * kPartials, (size_t)nb * kPartials * sizeof(double), "partial sums");
    });
    return hipSuccess;
}
hipError_t launch_fused_step(int prec, bool, const StepArgs& a, const StripItem* items, int w0, int nw, bool residual, hipStream_t)
{
    return step("march", prec, a, items, w0, nw, residual);
}
hipError_t launch_block_step(int prec, bool, const StepArgs& a, const StripItem* items, int w0, int nw, bool residual, hipStream_t)
{
    return step("block", prec, a, items, w0, nw, residual);
}
hipError_t launch_tile_step(int, int prec, bool, const StepArgs& a, const StripItem* items, int w0, int nw, bool residual,
                            hipStream_t)
{
    return step("tile", prec, a, items, w0, nw, residual);
}
hipError_t launch_reduce_partials(const double* partial, const int32_t* first, const int32_t* count, const CavityDesc* desc,
                                  int n_cav, double*, double* out, hipStream_t)
{
    submit([=] {
        check(desc, n_cav * sizeof(CavityDesc), "descriptors");
        check(out, n_cav * kResult * sizeof(double), "residual record");
        for (int c = 0; c < n_cav; ++c) {
            if (!inside(first + c, 4) || !inside(count + c, 4)) return fault("unit ranges");
            check(partial + (int64_t)first[c] * kPartials, (size_t)count[c] * kPartials * sizeof(double), "partial sums");
            double* o = out + c * kResult;
            const bool done = c < (int)converged.size() && converged[c];
            for (int q = 0; q < kResult; ++q) o[q] = 0.0;
            o[1] = o[3] = o[8] = 1.0;
            if (!done) o[0] = o[2] = o[7] = 1.0;
        }
    });
    return hipSuccess;
}
hipError_t launch_init(int, void*, void*, const CavityDesc*, const NodeBlock*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_fields(int, const void*, const CavityDesc*, int, const CavityDesc&, void*, void*, void*, int, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_state_out(int, const void*, const void*, const CavityDesc&, double, double*, double*, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_state_in(int, void*, void*, const CavityDesc&, double, const double*, const double*, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_energy(int, const void*, const CavityDesc*, const double*, int, const CavityDesc&, double*, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_probe(int, const void*, const CavityDesc*, int, const NodeBlock*, int, double*, const int32_t*, const int32_t*,
                        double*, uint32_t*, int, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_round_stochastic(const double*, const uint32_t*, float*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_power_law(const double*, double, double*, int64_t, hipStream_t) { return hipSuccess; }

hipError_t tangent_kinetic_energy(int, int, double, double, double, double, double, double, double, int, int64_t, hipStream_t,
                                  double*, double*, std::string&, bool)
{
    return hipSuccess;
}
size_t tangent_workspace_elems(int, int) { return 0; }
size_t tangent_scratch_capacity_elems() { return 0; }

struct AdjointSweep::Impl {
    size_t nn = 0;
};
AdjointSweep::AdjointSweep() : d(new Impl) {}
AdjointSweep::~AdjointSweep() { delete d; }
size_t AdjointSweep::work_doubles(const CavityDesc& c) { return 20 * (size_t)c.nx * c.ny; }
hipError_t AdjointSweep::init(const CavityDesc& c, int, double* work, hipStream_t)
{
    d->nn = (size_t)c.nx * c.ny;
    check(work, 20 * d->nn * sizeof(double), "adjoint work");
    return hipSuccess;
}
hipError_t AdjointSweep::objective(const double* state, hipStream_t)
{
    check(state, 10 * d->nn * sizeof(double), "final state");
    return hipSuccess;
}
hipError_t AdjointSweep::step_back(const void* f, const void* l, const void* f1, hipStream_t)
{
    check(f, 1, "trajectory");
    check(l, 1, "trajectory");
    check(f1, 1, "trajectory");
    return hipSuccess;
}
hipError_t AdjointSweep::finish(const CavityDesc&, double, double, double, double, hipStream_t, double* J, double grad[3])
{
    *J = grad[0] = grad[1] = grad[2] = 0.0;
    return hipSuccess;
}

}  // namespace ifd
