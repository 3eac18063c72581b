// wd_apply_noalloc: the operator application of wd_apply for callers that cannot allocate device
// memory (code under HIP graph capture, tight serving loops, harnesses that forbid allocation).
//
// wd_apply runs one kernel on the caller's fields and allocates only where the input overlaps the
// output (a copy of the input, kept by the handle). This variant keeps that copy in `scratch`, a fixed
// file-scope device array (one per GPU, held until the process ends), so it calls no hipMalloc, hipFree,
// pinned-memory allocation or host-to-device copy. The kernel and its launch configuration are those
// of wd_apply, so the results are bitwise the same.
//
// Host code never uses the name `scratch` as an address: on first use on a device (that device
// current) hipGetSymbolAddress gives the device address, kept per device, and only that address is
// passed to kernels. Every call on one GPU shares that GPU's array: calls that overlap on one GPU
// race (serialise them, e.g. on one stream).
#include <mutex>

#include "wd_host.hpp"

namespace wd {

static __device__ __align__(256) char scratch[kNoallocScratchBytes];

static std::mutex g_scratch_mu;
static char* g_scratch_addr[kNoallocMaxDevices];

// the device address of `scratch` on the current device
static char* scratch_address()
{
    int dev = 0;
    WD_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kNoallocMaxDevices) throw Error{WD_ERR_ARG, "device index out of range"};
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void* p = nullptr;
        WD_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) throw Error{WD_ERR_HIP, "hipGetSymbolAddress returned no address for the scratch array"};
        g_scratch_addr[dev] = (char*)p;
    }
    return g_scratch_addr[dev];
}

void apply_noalloc(wd_gauge* g, double kappa, double* out, const double* in, bool dag, hipStream_t s)
{
    if (g->geo.stride > kNoallocMaxStride)
        throw Error{WD_ERR_ARG, "lattice too large for wd_apply_noalloc: " + std::to_string(g->geo.stride) +
                                    " sites per parity, at most " + std::to_string(kNoallocMaxStride)};
    const size_t bytes = (size_t)g->V * 24 * sizeof(double);
    if (ranges_overlap(out, in, bytes)) {
        char* copy = scratch_address();
        WD_CHECK_HIP(hipMemcpyAsync(copy, in, bytes, hipMemcpyDeviceToDevice, s));
        in = (const double*)copy;
    }
    run_apply(g, kappa, out, in, dag, s);
}

} // namespace wd
