// Instantiations and launcher of the hop for small launches (k_hop_split in wd_hop.hpp).
#include "wd_hop.hpp"

namespace wd {

int split_blocks(int Vh) { return (Vh + SPLIT_SITES - 1) / SPLIT_SITES; }

#define SPLIT_CASE(SF_, LF_, DAG_, RED_)                                                                           \
    if (sf == SF_ && lf == LF_ && dag == DAG_ && red == RED_) {                                                    \
        if (tg) hipExtLaunchKernelGGL((k_hop_split<SF_, LF_, DAG_, RED_, !DAG_>), grid1(nblocks),                  \
                                      dim3(SPLIT_THREADS), 0, s, ev0, ev1, 0, jobs, njobs, sys, gated, exec);      \
        else hipExtLaunchKernelGGL((k_hop_split<SF_, LF_, DAG_, RED_, false>), grid1(nblocks),                     \
                                   dim3(SPLIT_THREADS), 0, s, ev0, ev1, 0, jobs, njobs, sys, gated, exec);         \
        return hipGetLastError();                                                                                  \
    }
#define SPLIT_FWD(SF_, LF_)                                                                                        \
    SPLIT_CASE(SF_, LF_, false, RED_NONE) SPLIT_CASE(SF_, LF_, false, RED_NORM)                                    \
    SPLIT_CASE(SF_, LF_, false, RED_ZDOT) SPLIT_CASE(SF_, LF_, false, RED_OUTX)
#define SPLIT_ALL(SF_, LF_)                                                                                        \
    SPLIT_FWD(SF_, LF_) SPLIT_CASE(SF_, LF_, true, RED_NONE) SPLIT_CASE(SF_, LF_, true, RED_ZDOT)

hipError_t launch_hop_split(int sf, int lf, bool dag, int red, const HopJob* jobs, int njobs, long nblocks,
                            SysState* sys, int gated, hipStream_t s, int* exec, int tg, hipEvent_t ev0, hipEvent_t ev1)
{
    if (tg && dag) return hipErrorInvalidValue;  // the adjoint hop runs on the caller's links only
    if (nblocks <= 0) return hipSuccess;
    SPLIT_ALL(SF32, L32_12) SPLIT_ALL(SF32, L16_12) SPLIT_ALL(SF32, LB16_12) SPLIT_ALL(SF32, L16_8)
    SPLIT_ALL(SF16, L32_12) SPLIT_ALL(SF16, L16_12) SPLIT_ALL(SF16, LB16_12) SPLIT_ALL(SF16, L16_8)
    SPLIT_ALL(SF64, L64_18) SPLIT_CASE(SF64, L64_18, true, RED_NORM)
    SPLIT_ALL(SF64, L64_12) SPLIT_CASE(SF64, L64_12, true, RED_NORM)
    return hipErrorInvalidValue;
}

} // namespace wd
