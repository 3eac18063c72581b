// Instantiations and launcher of the single-system hop for FP64 spinors and links (kernel template
// in wd_hop.hpp): the reliable updates, b_prec, eq. eo3, BiCGstab-M and wd_apply.
#include "wd_hop.hpp"

namespace wd {

hipError_t launch_hop64(bool dag, int lf, int red, const HopJob* jobs, int njobs, long nblocks, SysState* sys,
                        int gated, hipStream_t s, int* exec, int stage, int tg, int ntl, hipEvent_t ev0,
                        hipEvent_t ev1)
{
    const int sf = SF64;
    if (stage < 0) stage = hop_stage64_default();
    const int stage64 = stage;
    HOP_REDS(SF64, L64_18, false)
    HOP_REDS(SF64, L64_12, false)
    HOP_DAG_64(L64_18)
    HOP_DAG_64(L64_12)
    return hipErrorInvalidValue;
}

// both parities in one launch (k_hop's FULL)
#define HOP_FULL(LF_, DAG_, RED_)                                                                                  \
    if (lf == LF_ && dag == DAG_ && red == RED_) {                                                                 \
        if (tg) hipExtLaunchKernelGGL((k_hop<SF64, LF_, DAG_, RED_, FIN_STORE, true, false, !DAG_, true>),         \
                                      grid1(nblocks), dim3(BLOCK), 0, s, ev0, ev1, 0, jobs, njobs, sys, gated, exec); \
        else hipExtLaunchKernelGGL((k_hop<SF64, LF_, DAG_, RED_, FIN_STORE, true, false, false, true>),            \
                                   grid1(nblocks), dim3(BLOCK), 0, s, ev0, ev1, 0, jobs, njobs, sys, gated, exec); \
        return hipGetLastError();                                                                                  \
    }
void full_tile(HopJob& j)
{
    const int slice = j.g.Xh * j.g.Y * j.g.Z;
    j.tb = slice % BLOCK == 0 ? 8 : 0;
    j.bps = slice / BLOCK;
}

hipError_t launch_hop_full(bool dag, int lf, int red, const HopJob* jobs, int njobs, long nblocks, SysState* sys,
                           int gated, hipStream_t s, int* exec, int tg, hipEvent_t ev0, hipEvent_t ev1)
{
    if (tg && dag) return hipErrorInvalidValue;  // the adjoint hop runs on the caller's links only
    if (nblocks <= 0) return hipSuccess;
    HOP_FULL(L64_18, false, RED_ZDOT)
    HOP_FULL(L64_18, false, RED_OUTX)
    HOP_FULL(L64_18, false, RED_FULL)
    HOP_FULL(L64_18, false, RED_NORM)
    HOP_FULL(L64_12, false, RED_ZDOT)
    HOP_FULL(L64_12, false, RED_OUTX)
    HOP_FULL(L64_12, false, RED_FULL)
    HOP_FULL(L64_12, false, RED_NORM)
    return hipErrorInvalidValue;
}

} // namespace wd
