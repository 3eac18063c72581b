// A stand-in for the device, for tests of the library's host code without a GPU (tests/test_host_driver.py):
// the HIP calls and kernel launchers that wd_runtime.cpp, wd_solve.cpp and wd_api.cpp use, linked with those
// files into one library.
//
// Device memory is host memory, with a capacity, and every copy and fill is checked against the
// allocation it touches. Launches and asynchronous copies are queued; looking at the stream (hipStreamQuery)
// runs a few of them, waiting for it runs all. Kernels compute nothing but the systems' records: a
// script decides how each iteration and each FP64 update of the even-odd solver ends, and the record
// moves on as the finishers of wd_kernels.hip move it, reports to the host included.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <random>

#include "wd_host.hpp"

using namespace wd;

namespace {

struct Fake {
    std::map<char*, size_t> mem;
    size_t capacity = ~(size_t)0, live = 0, peak = 0;
    int out_of_range = 0;
    std::deque<std::function<void()>> queue;
    hipError_t error = hipSuccess;  // of a kernel that failed: what every later wait returns
    bool fail_unpack = false;
    int eager = 8;  // a look at the stream runs 0 .. eager queued operations
    std::mt19937 rng;
    double p_reliable = 0, p_converged = 1, p_verified = 1, p_breakdown = 0, p_nan = 0, bb = 1;
    bool ignore_maxit = false;
} F;

bool roll(double p) { return std::uniform_real_distribution<double>(0, 1)(F.rng) < p; }
void drain()
{
    while (!F.queue.empty()) {
        auto f = std::move(F.queue.front());
        F.queue.pop_front();
        f();
    }
}
hipError_t later(std::function<void()> f = [] {})
{
    F.queue.push_back(std::move(f));
    return hipSuccess;
}
// is [p, p + n) inside one allocation, or no device memory at all
bool in_range(const void* p, size_t n)
{
    auto it = F.mem.upper_bound((char*)p);
    if (it == F.mem.begin()) return true;
    --it;
    if ((char*)p >= it->first + it->second) return true;
    if ((char*)p + n <= it->first + it->second) return true;
    F.out_of_range++;
    return false;
}

void tell(SysState* S, double rr)
{
    if (!S->report) return;
    S->report->rr = rr;
    S->report->state = ((unsigned long long)S->status << 56) | ((unsigned long long)(S->nrel & 0xffffff) << 32) | (unsigned)S->iter;
}
bool open_gate(const SysState& S, int gated) { return !gated || ((gated >> S.status) & 1); }

void break_down(SysState* S)
{
    if (!roll(F.p_breakdown)) return;
    S->status = ST_BREAKDOWN;
    tell(S, S->rr);
}
void end_of_iteration(SysState* S)
{
    S->iter++;
    S->fresh = 0;
    S->rr *= 0.5;
    S->status = ST_RUNNING;
    if (roll(F.p_nan)) S->status = ST_NAN;
    else if (roll(F.p_converged)) S->status = ST_CONVERGED;
    else if (S->mixed && roll(F.p_reliable)) S->status = ST_RELIABLE;
    else if (!F.ignore_maxit && S->iter >= S->maxit) S->status = ST_MAXIT;
    tell(S, S->rr);
}
void end_of_update(SysState* S)
{
    const int was = S->status;
    const bool ok = roll(F.p_verified);
    const double rr = ok ? 0.0 : 0.25 * S->rr;
    S->nrel++;
    S->rr_true = rr;
    S->fresh = 1;
    S->t_zero = 0;
    if (ok && was != ST_RELIABLE && was != ST_BREAKDOWN) S->status = ST_DONE;
    else if (was == ST_MAXIT || (!F.ignore_maxit && S->iter >= S->maxit)) S->status = ST_NOCONV;
    else if (was == ST_BREAKDOWN) S->status = ++S->restarts > 2 ? ST_BROKEN : ST_SEL2;
    else S->status = S->dc ? ST_SEL2 : ST_SEL1;
    if (((GATE_GOES_ON >> was) & 1) && (S->status == ST_SEL1 || S->status == ST_SEL2)) {
        S->rr = rr + 1e-3;
        S->status = ST_RUNNING;
    }
    tell(S, S->status == ST_RUNNING ? S->rr : rr);
}

} // namespace

// ---------------------------------------------------------------- HIP
extern "C" {
hipError_t hipMalloc(void** p, size_t n)
{
    if (F.live + n > F.capacity) return hipErrorOutOfMemory;
    *p = std::calloc(1, n);
    F.mem[(char*)*p] = n;
    F.live += n;
    F.peak = std::max(F.peak, F.live);
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    drain();
    auto it = F.mem.find((char*)p);
    if (it == F.mem.end()) return hipErrorInvalidValue;
    F.live -= it->second;
    F.mem.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free, size_t* total)
{
    *total = F.capacity;
    *free = F.capacity - std::min(F.capacity, F.live);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    std::free(p);
    return hipSuccess;
}
// fields need no contents here: only small buffers (records, tables, partial sums) are written
static void fill(void* p, int v, size_t n)
{
    if (n < ((size_t)1 << 16)) std::memset(p, v, n);
}
hipError_t hipMemset(void* p, int v, size_t n)
{
    if (!in_range(p, n)) return hipErrorInvalidValue;
    drain();
    fill(p, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t)
{
    if (!in_range(p, n)) return hipErrorInvalidValue;
    return later([=] { fill(p, v, n); });
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    if (!in_range(d, n) || !in_range(s, n)) return hipErrorInvalidValue;
    drain();
    std::memcpy(d, s, n);
    return F.error;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    if (!in_range(d, n) || !in_range(s, n)) return hipErrorInvalidValue;
    return later([=] { std::memcpy(d, s, n); });
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    drain();
    return F.error;
}
hipError_t hipDeviceSynchronize()
{
    drain();
    return F.error;
}
hipError_t hipStreamQuery(hipStream_t)
{
    for (int k = (int)(F.rng() % (unsigned)(F.eager + 1)); k > 0 && !F.queue.empty(); k--) {
        auto f = std::move(F.queue.front());
        F.queue.pop_front();
        f();
    }
    if (F.error != hipSuccess) return F.error;
    return F.queue.empty() ? hipSuccess : hipErrorNotReady;
}
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600*, int) { return hipErrorNotSupported; }
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetLastError() { return hipSuccess; }
static char g_event;
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    *e = (hipEvent_t)&g_event;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t)
{
    drain();
    return F.error;
}
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t)
{
    *t = 0.f;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipErrorNotSupported; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipErrorNotSupported; }

// ---------------------------------------------------------------- control
void fake_reset(size_t capacity, unsigned seed)
{
    F.capacity = capacity;
    F.peak = F.live;
    F.out_of_range = 0;
    F.error = hipSuccess;
    F.fail_unpack = false;
    F.ignore_maxit = false;
    F.rng.seed(seed);
    F.p_reliable = F.p_breakdown = F.p_nan = 0;
    F.p_converged = F.p_verified = F.bb = 1;
}
void fake_script(double reliable, double converged, double verified, double breakdown, double nan)
{
    F.p_reliable = reliable;
    F.p_converged = converged;
    F.p_verified = verified;
    F.p_breakdown = breakdown;
    F.p_nan = nan;
}
void fake_ignore_maxit() { F.ignore_maxit = true; }
void fake_fail_unpack() { F.fail_unpack = true; }
size_t fake_live() { return F.live; }
size_t fake_peak() { return F.peak; }
int fake_out_of_range() { return F.out_of_range; }
}

// ---------------------------------------------------------------- kernels
namespace wd {

static hipError_t ran(int* exec, int n)
{
    return later([=] {
        if (exec) *exec += n;
    });
}
hipError_t launch_hop(int, int, bool, int, int, const HopJob*, int njobs, long, SysState*, int, hipStream_t, int* exec, int,
                      int, int, hipEvent_t, hipEvent_t)
{
    return ran(exec, njobs);
}
hipError_t launch_hop_full(int, int, const HopJob*, int njobs, long, SysState*, int, hipStream_t, int* exec, int,
                           hipEvent_t, hipEvent_t)
{
    return ran(exec, njobs);
}
hipError_t launch_hop_split(int, int, bool, int, const HopJob*, int njobs, long, SysState*, int, hipStream_t, int* exec,
                            int, hipEvent_t, hipEvent_t)
{
    return ran(exec, njobs);
}
hipError_t launch_hop_mrhs(int, int, bool, int, int, const HopJob*, int njobs, long, SysState*, int, hipStream_t,
                           int* exec, hipEvent_t, hipEvent_t)
{
    return ran(exec, njobs);
}
hipError_t launch_update(int, int, int, const HopJob*, int njobs, long, SysState*, int, hipStream_t, int* exec, int, int,
                         int, hipEvent_t, hipEvent_t)
{
    return ran(exec, njobs);
}
// The systems of one launch move on one by one, in any order: the host may look between them.
template <class J, class Fn>
static void each_system(const J* jobs, int n, Fn fn)
{
    std::vector<int> order(n);
    for (int i = 0; i < n; i++) order[i] = i;
    std::shuffle(order.begin(), order.end(), F.rng);
    for (int i : order) later([=] { fn(jobs[i].sys); });
}
hipError_t launch_finish(int, int fin, const FinJob* fins, int nfin, SysState* sys, int gated, hipStream_t, hipEvent_t,
                         hipEvent_t)
{
    each_system(fins, nfin, [=](int i) {
        SysState* S = sys + i;
        if (!open_gate(*S, gated)) return;
        if (fin == FIN_STORE) {
            S->red[2] = F.bb;
        } else if (fin == FIN_RESTART) {
            S->rr = S->maxrr = S->rr > 0 ? S->rr : 1.0;
            S->red[2] = F.bb;
            S->status = ST_RUNNING;
            tell(S, S->rr);
        } else if (fin == FIN_CHIALPHA) {
            break_down(S);
        } else if (fin == FIN_RR || fin == FIN_CGB) {
            end_of_iteration(S);
        } else if (fin == FIN_UPDATE) {
            end_of_update(S);
        }
    });
    return hipSuccess;
}
hipError_t launch_sweep(int op, int, const SweepJob* jobs, int njobs, long, SysState* sys, int gated, hipStream_t, int* exec,
                        hipEvent_t, hipEvent_t, bool fold)
{
    (void)ran(exec, njobs);
    if (fold && (op == OP_XR || op == OP_S))
        each_system(jobs, njobs, [=](int i) {
            if (!open_gate(sys[i], gated)) return;
            if (op == OP_XR) break_down(sys + i);
            else end_of_iteration(sys + i);
        });
    return hipSuccess;
}
hipError_t launch_shift_coef(bool, ShiftBlock*, ShiftScal*, const SpinorRef*, ShiftCoef*, int, const SysState*, hipStream_t)
{
    return later();
}
hipError_t launch_shift_update(int, const ShiftVectors&, long, const ShiftBlock*, const ShiftCoef*, hipStream_t, int* exec,
                               hipEvent_t, hipEvent_t)
{
    return ran(exec, 1);
}
static hipError_t unpack()
{
    return later([] {
        if (F.fail_unpack) F.error = hipErrorLaunchFailure;
    });
}
hipError_t launch_unpack_spinor(int, double*, const Geo&, SpinorRef, SpinorRef, int, double, hipStream_t, const double*, int)
{
    return unpack();
}
hipError_t launch_unpack_eo(double*, const Geo&, SpinorRef, SpinorRef, SpinorRef, SpinorRef, double, double, int, double,
                            hipStream_t, const double*, int)
{
    return unpack();
}
hipError_t launch_pack_spinor(int, const double*, const Geo&, SpinorRef, SpinorRef, int, double, hipStream_t, const double*, int)
{
    return later();
}
hipError_t launch_pack_links(const double*, const Geo&, void*, void*, long, hipStream_t) { return later(); }
hipError_t launch_convert_links(int, int, const void*, void*, int, long, hipStream_t) { return later(); }
hipError_t launch_temporal_gauge(const double*, const Geo&, double*, double*, hipStream_t) { return later(); }
hipError_t launch_recon_check(const void*, int Vh, long, double* blockmax, hipStream_t, int)
{
    return later([=] { std::memset(blockmax, 0, sizeof(double) * ((Vh + BLOCK - 1) / BLOCK)); });
}
hipError_t launch_apply(bool, double*, const double*, const Geo&, const void*, const void*, long, double, hipStream_t,
                        hipEvent_t, hipEvent_t)
{
    return later();
}
hipError_t launch_guess(const GuessArgs&, hipStream_t) { return later(); }
hipError_t launch_dots(SpinorRef, const SpinorRef*, int, const Geo&, double*, double*, hipStream_t) { return later(); }
hipError_t launch_grad(const double*, const double*, const Geo&, const void*, const void*, long, double*, int, hipStream_t)
{
    return later();
}
int mrhs_kt(int k) { return k <= 2 ? 2 : k <= 4 ? 4 : 0; }
int split_blocks(int Vh) { return (Vh + 63) / 64; }
void full_tile(HopJob& j) { j.tb = j.bps = 0; }
void apply_noalloc(wd_gauge*, double, double*, const double*, bool, hipStream_t) {}

} // namespace wd
