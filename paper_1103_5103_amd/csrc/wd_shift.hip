// The shifted systems of BiCGstab-M (Sec. 6.1) and CG-M, brought up to date once per block of
// iterations.
//
// Per iteration the shifted updates are
//   BiCGstab-M: x^s <- x^s - beta^s s^s + chi^s rho_n zeta_{n+1} w
//               s^s <- zeta_{n+1} rho_{n+1} r_{n+1}
//                      + alpha^s (s^s - (chi^s / beta^s) rho_n (zeta_{n+1} w - zeta_n r_n))
//   CG-M:       x^s <- x^s + alpha^s p^s,  p^s <- zeta_{n+1} r_{n+1} + beta^s p^s
// so over m iterations x^s and s^s (p^s) are linear combinations of their old values and of the base
// system's r_0, w_0, r_1, ..., r_m, with coefficients that follow from the scalars alone. Applied one
// iteration at a time they move 4 spinors per shift and iteration, the bulk of a multi-shift solve;
// applied to a block they move (4 k + 2 m + 1) / m spinors per iteration for k shifts (CG-M
// (4 k + m) / m), against 4 k + 2 (4 k) before. The price is m + 1 residuals (and m vectors w) kept
// instead of 2 (1), and more arithmetic, 8 m complex multiply-adds per number, shift and block, still
// far below the memory time.
#include "wd_hop.hpp"

namespace wd {

__device__ __forceinline__ cx<double> c64(double2 a) { return {a.x, a.y}; }
__device__ __forceinline__ double2 d64(cx<double> a) { return make_double2(a.re, a.im); }
__device__ __forceinline__ cx<double> cdivide(cx<double> a, cx<double> b)
{
    const double d = b.re * b.re + b.im * b.im;
    return {(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}

// One wavefront: lane q runs shift q's recurrences over the block's iterations and forms its
// coefficients; the shifts that were active are packed into coef[0 .. nrun).
template <bool CG>
__global__ __launch_bounds__(64) void k_shift_coef(ShiftBlock* __restrict__ B, ShiftScal* __restrict__ sh,
                                                   const SpinorRef* __restrict__ sv, ShiftCoef* __restrict__ coef,
                                                   int ns, const SysState* __restrict__ base)
{
    __shared__ cx<double> sx[32][SHIFT_NB + 1], ss[32][SHIFT_NB + 1];
    const int q = threadIdx.x, cnt = B->count;
    const bool first = B->updates == 0;
    const double target2 = B->target2;
    if (cnt == 0 && !first) {
        if (q == 0) B->nrun = -1;
        return;
    }
    const int it0 = base->iter - cnt;  // iterations before the block
    const bool run = q < ns && (sh[q].active || first);
    bool store_s = false;
    if (run) {
        ShiftScal z = sh[q];
        cx<double>*X = sx[q], *S = ss[q];
        for (int k = 0; k <= SHIFT_NB; k++) X[k] = S[k] = cx<double>{0.0, 0.0};
        S[first ? 1 : 0] = cx<double>{1.0, 0.0};  // the first block starts from s = r_0, x = 0
        const cx<double> one = {1.0, 0.0};
        const int nv = CG ? cnt + 1 : 2 * cnt + 1;
        cx<double> ap = c64(B->alpha_prev), bp = c64(B->beta_prev);
        for (int i = 0; i < cnt && z.active; i++) {
            const IterScal I = B->it[i];
            const cx<double> zp = c64(z.zeta_prev), ze = c64(z.zeta);
            cx<double> zn;
            double rz2;  // |r^s|^2 / |r|^2 after the iteration
            if constexpr (CG) {
                // base: alpha_n, beta_{n+1}; alpha_{n-1} (ap) and beta_n (bp)
                const double a = I.alpha.x;
                const double den = zp.re * ap.re * (1.0 + a * z.sigma) + a * bp.re * (zp.re - ze.re);
                zn = {ze.re * zp.re * ap.re / den, 0.0};
                const double as = a * zn.re / ze.re, g = zn.re / ze.re, bs = I.beta.x * g * g;
                for (int k = 0; k <= nv; k++) {
                    X[k] = X[k] + as * S[k];
                    S[k] = bs * S[k];
                }
                S[2 + i] = S[2 + i] + zn;
                rz2 = zn.re * zn.re;
                z.active = !(rz2 * I.rr <= target2);
                ap = c64(I.alpha);
                bp = c64(I.beta);
            } else {
                const cx<double> be = c64(I.beta), ch = c64(I.chi), al = c64(I.alpha), rho = c64(z.rho);
                // zeta_{n+1} and beta^s from the collinearity of the residuals
                const cx<double> den = be * ap * (zp - ze) + zp * bp * (one - z.sigma * be);
                zn = cdivide(ze * zp * bp, den);
                const cx<double> bs = cdivide(be * zn, ze);
                const cx<double> d = one + z.sigma * ch;
                const cx<double> cs = cdivide(ch, d), rn = cdivide(rho, d);
                // alpha^s_{n+1} = alpha_{n+1} zeta_{n+1} beta^s_n / (zeta_n beta_n)
                const cx<double> as = cdivide(al * zn * bs, ze * be);
                const cx<double> cb = cdivide(cs, bs) * rho;
                for (int k = 0; k <= nv; k++) {
                    X[k] = X[k] - bs * S[k];
                    S[k] = as * S[k];
                }
                X[2 + 2 * i] = X[2 + 2 * i] + cs * rho * zn;           // w_i
                S[1 + 2 * i] = S[1 + 2 * i] + as * cb * ze;            // r_i
                S[2 + 2 * i] = S[2 + 2 * i] - as * cb * zn;            // w_i
                S[3 + 2 * i] = S[3 + 2 * i] + zn * rn;                 // r_{i+1}
                const cx<double> zr = zn * rn;
                rz2 = zr.re * zr.re + zr.im * zr.im;
                z.active = !(rz2 * I.rr < target2);
                z.rho = d64(rn);
                ap = al;
                bp = be;
            }
            z.zeta_prev = z.zeta;
            z.zeta = d64(zn);
            if (!z.active) z.conv_iter = it0 + i + 1;
        }
        sh[q] = z;
        store_s = z.active != 0;
    }
    const unsigned long long m = __ballot(run);
    if (run) {
        ShiftCoef& C = coef[__popcll(m & ((1ull << q) - 1))];
        C.x = sv[2 * q].p;
        C.s = sv[2 * q + 1].p;
        C.store_s = store_s;
        for (int k = 0; k <= SHIFT_NB; k++) {
            C.cx[k] = d64(sx[q][k]);
            C.cs[k] = d64(ss[q][k]);
        }
    }
    __syncthreads();
    if (q == 0) {
        B->nrun = __popcll(m);
        B->first = first;
        // a block without iterations (the solve stopped in its first one) writes x = 0
        B->mask = cnt == 0 ? 0u : CG ? ((1u << (cnt + 1)) - 1u) & ~(first ? 0u : 1u) : (1u << (2 * cnt + 1)) - 1u;
        if (cnt > 0) {
            B->alpha_prev = B->it[cnt - 1].alpha;
            B->beta_prev = B->it[cnt - 1].beta;
        }
        B->count = 0;
        B->updates += 1;
    }
}

// The update: one thread per complex number of the fields (they share one layout, so it is
// elementwise and fully coalesced). The block vectors stay in registers for all shifts; the
// coefficients are wave-uniform. Bound by memory (about 5.4 TB/s at 32^3x64): the next shift's x and
// s are loaded before the present one's sums.
template <int NB>
__global__ __launch_bounds__(BLOCK) void k_shift_update(ShiftVectors V, long n, const ShiftBlock* __restrict__ B,
                                                        const ShiftCoef* __restrict__ coef, int* exec)
{
    const int nrun = B->nrun;
    if (nrun <= 0) return;
    if (exec && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(exec, 1);
    const long e = (long)blockIdx.x * BLOCK + threadIdx.x;
    if (e >= n) return;
    const unsigned mask = B->mask;
    const bool first = B->first != 0;
    d2v b[NB];
#pragma unroll
    for (int k = 0; k < NB; k++) {
        b[k] = d2v{0.0, 0.0};
        if ((mask >> k) & 1) b[k] = gldt<d2v, true>(V.v[k], e);
    }
    d2v x = {0.0, 0.0}, s = {0.0, 0.0};
    if (!first) {
        x = gldt<d2v, true>(coef[0].x, e);
        s = gldt<d2v, true>(coef[0].s, e);
    }
    for (int i = 0; i < nrun; i++) {
        const ShiftCoef& C = coef[i];
        d2v xn = {0.0, 0.0}, sn = {0.0, 0.0};
        if (!first && i + 1 < nrun) {
            xn = gldt<d2v, true>(coef[i + 1].x, e);
            sn = gldt<d2v, true>(coef[i + 1].s, e);
        }
        auto mad = [](d2v a, double2 c, d2v v) {
            a[0] = fma(c.x, v[0], a[0]);
            a[1] = fma(c.x, v[1], a[1]);
            a[0] = fma(-c.y, v[1], a[0]);
            a[1] = fma(c.y, v[0], a[1]);
            return a;
        };
        x = mad(x, C.cx[0], s);
        s = mad(d2v{0.0, 0.0}, C.cs[0], s);
#pragma unroll
        for (int k = 0; k < NB; k++)
            if ((mask >> k) & 1) {
                x = mad(x, C.cx[1 + k], b[k]);
                s = mad(s, C.cs[1 + k], b[k]);
            }
        gst<d2v, true>(C.x, e, x);
        if (C.store_s) gst<d2v, true>(C.s, e, s);
        x = xn;
        s = sn;
    }
}

hipError_t launch_shift_coef(bool cg, ShiftBlock* blk, ShiftScal* sh, const SpinorRef* sv, ShiftCoef* coef, int ns,
                             const SysState* base, hipStream_t s)
{
    if (ns < 1 || ns > 32) return hipErrorInvalidValue;
    if (cg) hipLaunchKernelGGL((k_shift_coef<true>), dim3(1), dim3(64), 0, s, blk, sh, sv, coef, ns, base);
    else hipLaunchKernelGGL((k_shift_coef<false>), dim3(1), dim3(64), 0, s, blk, sh, sv, coef, ns, base);
    return hipGetLastError();
}

hipError_t launch_shift_update(int nb, const ShiftVectors& v, long n, const ShiftBlock* blk, const ShiftCoef* coef,
                               hipStream_t s, int* exec, hipEvent_t ev0, hipEvent_t ev1)
{
    constexpr int NBC = SHIFT_BLOCK + 1;  // CG-M: r_0 .. r_m
    if (nb > SHIFT_NB || n <= 0) return hipErrorInvalidValue;
    const dim3 grid = grid1((n + BLOCK - 1) / BLOCK);
    if (nb <= NBC)
        hipExtLaunchKernelGGL((k_shift_update<NBC>), grid, dim3(BLOCK), 0, s, ev0, ev1, 0, v, n, blk, coef, exec);
    else
        hipExtLaunchKernelGGL((k_shift_update<SHIFT_NB>), grid, dim3(BLOCK), 0, s, ev0, ev1, 0, v, n, blk, coef, exec);
    return hipGetLastError();
}

} // namespace wd
