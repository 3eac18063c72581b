// Instantiations and launcher of the single-system hop for FP64 spinors and links (kernel template
// in wd_hop.hpp): 1/2 D_eo b_o, the start residual, eq. eo3, CG's operator, and (full lattice) BiCGstab-M.
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
#define HOP_FULL(LF_, RED_)                                                                                        \
    if (lf == LF_ && red == RED_) {                                                                                \
        if (tg) hipExtLaunchKernelGGL((k_hop<SF64, LF_, false, RED_, FIN_STORE, true, false, true, true>),         \
                                      grid1(nblocks), dim3(BLOCK), 0, s, ev0, ev1, 0, jobs, njobs, sys, gated, exec); \
        else hipExtLaunchKernelGGL((k_hop<SF64, LF_, false, RED_, FIN_STORE, true, false, false, true>),           \
                                   grid1(nblocks), dim3(BLOCK), 0, s, ev0, ev1, 0, jobs, njobs, sys, gated, exec); \
        return hipGetLastError();                                                                                  \
    }
void full_tile(HopJob& j)
{
    const int slice = j.g.Xh * j.g.Y * j.g.Z;
    j.tb = slice % BLOCK == 0 ? 8 : 0;
    j.bps = slice / BLOCK;
}

hipError_t launch_hop_full(int lf, int red, const HopJob* jobs, int njobs, long nblocks, SysState* sys,
                           int gated, hipStream_t s, int* exec, int tg, hipEvent_t ev0, hipEvent_t ev1)
{
    if (nblocks <= 0) return hipSuccess;
    HOP_FULL(L64_18, RED_ZDOT)
    HOP_FULL(L64_18, RED_OUTX)
    HOP_FULL(L64_18, RED_FULL)
    HOP_FULL(L64_18, RED_NORM)
    HOP_FULL(L64_12, RED_ZDOT)
    HOP_FULL(L64_12, RED_OUTX)
    HOP_FULL(L64_12, RED_FULL)
    HOP_FULL(L64_12, RED_NORM)
    return hipErrorInvalidValue;
}

} // namespace wd
