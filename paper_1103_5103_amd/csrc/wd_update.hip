// FP64 residual update of the even-odd solves (reliable updates and defect correction, Sec. 6.2.4):
//   x_hi <- x_hi + x_lo,  r = b_prec - M_prec x_hi  (FP64),  r_lo = r
// in two hops and one finisher:
//   first hop   T <- T + D_oe x_lo, where T holds D_oe x_hi (0 at the start without a start vector); where
//               it does not (the first update after a start vector that came with its residual)
//               T = D_oe (x_hi + x_lo), the sum formed as it is loaded;
//   second hop  r = b_prec - a^2 (x_hi + x_lo) + 1/4 D_eo T; its epilogue stores the new x_hi and, for a
//               system that goes on, brings s up to date (the s update of the iteration in which a
//               reliable update fell due was gated off) or restarts with rhat = s = r, stores r_lo, and
//               forms |r|^2, <rhat, r_lo>, |r_lo|^2. A system whose update only verifies convergence
//               leaves r in FP64 instead (HopJob::keep: every system does).
// All arithmetic is FP64. Against sweeps of their own for x_hi += x_lo and r_lo = r this saves both and,
// per site, 576 B of x and r traffic; x_lo is not cleared either (SysState::fresh: it counts as zero until
// it is written). Measured per update (x_hi += x_lo, two hops, r_lo = r before; two hops now), both bound by
// memory: 6 systems of 24^3x48, FP32 spinors 208 + 371 + 497 + 182 = 1258 -> 304 + 636 us; 96 systems (16^3x32 and
// smaller, FP16) 401 + 609 + 806 + 194 = 2010 -> 485 + 930 us; 8^4 (launches bound by latency) 32 -> 19 us.
#include "wd_hop.hpp"

namespace wd {

// keeps the next part's loads from being issued before this part is done (all at once they would spill)
__device__ __forceinline__ void part_done() { asm volatile("" ::: "memory"); }

// x_hi + x_lo of site cb, stored as the new x_hi
template <int SFL, bool NT>
__device__ __forceinline__ void update_x(const HopJob& J, const SysState* S, int cb, cx<double> xh[12])
{
    using T = typename SReal<SFL>::T;
    load_spinor<SF64, double, NT>(J.x1, cb, xh);
    if (S->fresh) return;
    cx<T> xl[12];
    load_spinor<SFL == SF64 ? SF64 : SF32, T, NT>(J.z, cb, xl);
#pragma unroll
    for (int k = 0; k < 12; k++) xh[k] = xh[k] + mk<double>((double)xl[k].re, (double)xl[k].im);
    store_spinor<SF64, double, NT>(J.x1, cb, xh);
}

// the second hop's epilogue on site cb; acc: r = b_prec - M_prec x
template <int SFL, bool NT>
__device__ __forceinline__ void update_residual(const HopJob& J, const SysState* S, int cb, const cx<double> acc[12],
                                                double v[NRED])
{
    using T = typename SReal<SFL>::T;
#pragma unroll
    for (int k = 0; k < 12; k++) v[2] += acc[k].re * acc[k].re + acc[k].im * acc[k].im;
    const int st = S->status;
    const bool on = (GATE_GOES_ON >> st) & 1;
    if (!on || J.keep) store_spinor<SF64, double, NT>(J.out, cb, acc);
    if (!on) return;
    const bool restart = S->dc || st == ST_BREAKDOWN;
    cx<T> r[12], q[12], rh[12];
    if (!restart && J.s_current) load_spinor<SFL, T, NT>(J.u_rh, cb, rh);
    else if (!restart) {
        // s <- r_{n+1} + alpha (s - chi A s) with the iterated residual, before it is replaced
        const cx<T> alpha = mk<T>((T)S->alpha.x, (T)S->alpha.y), chi = mk<T>((T)S->chi.x, (T)S->chi.y);
        cx<T> as[12];
        load_spinor<SFL, T, NT>(J.u_r, cb, r);
        load_spinor<SFL, T, NT>(J.u_s, cb, q);
        load_spinor<SFL, T, NT>(J.u_as, cb, as);
        load_spinor<SFL, T, NT>(J.u_rh, cb, rh);
#pragma unroll
        for (int k = 0; k < 12; k++) q[k] = r[k] + alpha * (q[k] - chi * as[k]);
        store_spinor<SFL, T>(J.u_s, cb, q);
    }
#pragma unroll
    for (int k = 0; k < 12; k++) r[k] = mk<T>((T)acc[k].re, (T)acc[k].im);
    store_spinor<SFL, T, NT>(J.u_r, cb, r);
    as_stored<SFL, T>(r);
    if (restart) {
        store_spinor<SFL, T, NT>(J.u_rh, cb, r);
        store_spinor<SFL, T>(J.u_s, cb, r);
#pragma unroll
        for (int k = 0; k < 12; k++) rh[k] = r[k];
    }
#pragma unroll
    for (int k = 0; k < 12; k++) {
        v[0] += (double)rh[k].re * r[k].re + (double)rh[k].im * r[k].im;
        v[1] += (double)rh[k].re * r[k].im - (double)rh[k].im * r[k].re;
        v[3] += (double)r[k].re * r[k].re + (double)r[k].im * r[k].im;
    }
}

// HOP 1: T += D_oe x_lo, SF = storage of x_lo. HOP 3: T = D_oe (x_hi + x_lo), SF = storage of x_lo. HOP 2: the
// second hop, SF = storage of the iteration. Launch shape, block order and link policy of k_hop in FP64.
template <int HOP, int SF> struct UpdIn {
    static constexpr int SFI = HOP == 1 ? SF : SF64;   // the hop's input
    static constexpr int SFA = HOP == 3 ? SF : -1;     // added to it
};

template <int HOP, int SF, int LF, bool TG, bool NTL>
__global__ __launch_bounds__(BLOCK) void k_update(const HopJob* __restrict__ jobs, int njobs,
                                                  SysState* __restrict__ sys, int gated, int* exec)
{
    constexpr int SFI = UpdIn<HOP, SF>::SFI, SFA = UpdIn<HOP, SF>::SFA;
    const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    int jx = find_job(jobs, njobs, b);
    int lb = b - jobs[jx].blk0;
    if (jobs[jx].ilv > 1) {
        const int K = jobs[jx].ilv;
        jx = jx - jobs[jx].ilv_pos + lb % K;
        lb /= K;
    }
    const HopJob& J = jobs[jx];
    SysState* S = sys + J.sys;
    if (!((gated >> S->status) & 1)) return;
    if (exec && lb == 0 && threadIdx.x == 0) atomicAdd(exec, 1);
    const int cb0 = tiled_block(J, lb) * BLOCK;
    const int cb = cb0 + threadIdx.x;
    const bool fresh = S->fresh != 0;
    if (HOP == 1 && fresh) {  // x_lo = 0: T stays
        if (S->t_zero && cb < J.g.Vh) {
            cx<double> zero[12];
#pragma unroll
            for (int k = 0; k < 12; k++) zero[k] = mk<double>(0.0, 0.0);
            store_spinor<SF64, double>(J.out, cb, zero);
        }
        return;
    }
    __shared__ Stg<SFI, true> stg;
    const int H = J.g.Xh <= STG_H_MAX ? J.g.Xh : 0;
    const int base = cb0 - H, nsl = BLOCK + 2 * H;
    const SpinorRef& in = HOP == 1 ? J.z : J.in;
    const SpinorRef* add = HOP == 3 && !fresh ? &J.z : nullptr;
    if constexpr (HOP == 3) {
        // the window holds sums: through registers
        for (int k = threadIdx.x; k < nsl; k += BLOCK) {
            const int i = base + k;
            if (i >= 0 && i < J.g.Vh) {
                cx<double> q[12];
                load_spinor_sum<SF64, SFA, double>(in, add, i, q);
#pragma unroll
                for (int j = 0; j < 12; j++) stg.c[j][k] = d2v{q[j].re, q[j].im};
            }
        }
    } else {
        stage_window<SFI>(stg, in, base, nsl, J.g.Vh);
        stage_wait();
    }
    __syncthreads();
    double v[NRED] = {};
    if (cb < J.g.Vh) {
        cx<double> acc[12];
        const HopIn<SFI, true, SFA> hin{in, stg, base, nsl, TG && J.tg != 0, J.nc != 0, nullptr, add};
        hop_site<false, SFI, LF, true, NTL, false, double>(J.g, J.parity, cb, hin, J.links, J.lcs, acc);
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = J.c2 * acc[k];
        if constexpr (HOP == 2) {
            cx<double> q[12];
            load_spinor<SF64, double, NTL>(J.x0, cb, q);
#pragma unroll
            for (int k = 0; k < 12; k++) acc[k] = acc[k] + J.c0 * q[k];
            part_done();
            update_x<SF, NTL>(J, S, cb, q);
#pragma unroll
            for (int k = 0; k < 12; k++) acc[k] = acc[k] + J.c1 * q[k];
            part_done();
            update_residual<SF, NTL>(J, S, cb, acc, v);
        } else {
            if (HOP == 1 && !S->t_zero) {
                cx<double> q[12];
                load_spinor<SF64, double, NTL>(J.out, cb, q);
#pragma unroll
                for (int k = 0; k < 12; k++) acc[k] = acc[k] + q[k];
            }
            store_spinor<SF64, double, NTL>(J.out, cb, acc);
        }
    }
    if constexpr (HOP == 2) write_partials<4>(v, S, J.rblk0 + lb);
}

// The same for small launches, as k_hop_split.
template <int HOP, int SF, int LF, bool TG>
__global__ __launch_bounds__(SPLIT_THREADS) void k_update_split(const HopJob* __restrict__ jobs, int njobs,
                                                                SysState* __restrict__ sys, int gated, int* exec)
{
    constexpr int SFI = UpdIn<HOP, SF>::SFI, SFA = UpdIn<HOP, SF>::SFA;
    __shared__ d2v part[7][12][SPLIT_SITES];
    const int b = (int)blockIdx.x;
    const HopJob& J = jobs[find_job(jobs, njobs, b)];
    SysState* S = sys + J.sys;
    if (!((gated >> S->status) & 1)) return;
    const int lb = b - J.blk0;
    if (exec && lb == 0 && threadIdx.x == 0) atomicAdd(exec, 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
    const int cb = lb * SPLIT_SITES + lane;
    const bool ok = cb < J.g.Vh;
    const bool fresh = S->fresh != 0, t_zero = S->t_zero != 0;
    if (wave < 4) {
        const Stg<SFI, false> none{};
        const SpinorRef* add = HOP == 3 && !fresh ? &J.z : nullptr;
        const HopIn<SFI, false, SFA> hin{HOP == 1 ? J.z : J.in, none, 0, 0, TG && J.tg != 0, J.nc != 0, nullptr, add};
        split_part<false, LF, double>(J, hin, wave, lane, cb, ok && !(HOP == 1 && fresh), part);
        __syncthreads();
        return;
    }
    cx<double> p[12], q[12];
    if (ok) {
        if constexpr (HOP == 2) {
            load_spinor<SF64, double>(J.x0, cb, p);
            update_x<SF, false>(J, S, cb, q);
        } else if (HOP == 1 && !t_zero) {
            load_spinor<SF64, double>(J.out, cb, q);
        }
    }
    __syncthreads();
    double v[NRED] = {};
    if (ok) {
        cx<double> acc[12];
        split_sum<double>(part, lane, acc);
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = J.c2 * acc[k];
        if constexpr (HOP == 2) {
#pragma unroll
            for (int k = 0; k < 12; k++) acc[k] = acc[k] + J.c0 * p[k];
#pragma unroll
            for (int k = 0; k < 12; k++) acc[k] = acc[k] + J.c1 * q[k];
            part_done();
            update_residual<SF, false>(J, S, cb, acc, v);
        } else {
            if (HOP == 1 && !t_zero)
#pragma unroll
                for (int k = 0; k < 12; k++) acc[k] = acc[k] + q[k];
            store_spinor<SF64, double>(J.out, cb, acc);
        }
    }
    if constexpr (HOP == 2) {
        double* P = S->partials + (long)(J.rblk0 + lb) * NRED;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const double s = wave_sum(v[k]);
            if (lane == 0) P[k] = s;
        }
    }
}

#define UPDATE_LAUNCH(K_, THREADS_)                                                                                \
    hipExtLaunchKernelGGL(K_, grid1(nblocks), dim3(THREADS_), 0, s, ev0, ev1, 0, jobs, njobs, sys, gated, exec)
#define UPDATE_CASE(HOP_, SF_, LF_)                                                                                \
    if (hop == HOP_ && sf == SF_ && lf == LF_) {                                                                   \
        if (split && tg) UPDATE_LAUNCH((k_update_split<HOP_, SF_, LF_, true>), SPLIT_THREADS);                     \
        else if (split) UPDATE_LAUNCH((k_update_split<HOP_, SF_, LF_, false>), SPLIT_THREADS);                     \
        else if (tg && ntl) UPDATE_LAUNCH((k_update<HOP_, SF_, LF_, true, true>), BLOCK);                          \
        else if (tg) UPDATE_LAUNCH((k_update<HOP_, SF_, LF_, true, false>), BLOCK);                                \
        else if (ntl) UPDATE_LAUNCH((k_update<HOP_, SF_, LF_, false, true>), BLOCK);                               \
        else UPDATE_LAUNCH((k_update<HOP_, SF_, LF_, false, false>), BLOCK);                                       \
        return hipGetLastError();                                                                                  \
    }

hipError_t launch_update(int hop, int sf, int lf, const HopJob* jobs, int njobs, long nblocks, SysState* sys, int gated,
                         hipStream_t s, int* exec, int split, int tg, int ntl, hipEvent_t ev0, hipEvent_t ev1)
{
    if (nblocks <= 0) return hipSuccess;
    UPDATE_CASE(1, SF64, L64_18) UPDATE_CASE(1, SF64, L64_12) UPDATE_CASE(1, SF32, L64_18) UPDATE_CASE(1, SF32, L64_12)
    UPDATE_CASE(3, SF64, L64_18) UPDATE_CASE(3, SF64, L64_12) UPDATE_CASE(3, SF32, L64_18) UPDATE_CASE(3, SF32, L64_12)
    UPDATE_CASE(2, SF64, L64_18) UPDATE_CASE(2, SF64, L64_12) UPDATE_CASE(2, SF32, L64_18) UPDATE_CASE(2, SF32, L64_12)
    UPDATE_CASE(2, SF16, L64_18) UPDATE_CASE(2, SF16, L64_12)
    return hipErrorInvalidValue;
}

} // namespace wd
