// wd_apply / wd_apply_dag / wd_apply_noalloc: M(kappa) (Sec. 2, eq. 3 and 4) in FP64 straight from and
// to the caller's canonical fields, both parities in one launch, no packed copies.
//
// One wavefront per 64 consecutive canonical sites (one block). A site's spinor is 192 contiguous
// bytes, so lanes that load their own or their neighbour's spinor would touch 64 cache lines per
// instruction; instead the wave loads each of the seven runs of 64 sites that its stencil needs (its
// own, which also serves x +- 1, and the y, z, t neighbours of its first site) as contiguous 16-byte
// pieces and transposes them in LDS (13 pieces per site: no bank conflicts). Lanes whose neighbour is
// not in the run (periodic wraps inside it) load it from memory. The next run is loaded before the
// present direction's arithmetic; one buffer serves all runs (the own spinors, needed again at the end,
// are loaded again), which leaves 2 waves per SIMD, the limit of the registers. The output goes back
// through LDS the same way.
//
// Links: the 18-real internal format, forward slots only (the backward link of a site is its
// neighbour's forward one, which the wave next to it uses as well). Lanes 2 i and 2 i + 1 are the two
// sites of checkerboard index i, one of each parity, so a wave reads 512 contiguous bytes of either
// parity's array per piece.
//
// Blocks walk t fastest within groups of 64 blocks of a t-slice (32^3x64 in site order / groups of 16 /
// 32 / 64 / 128: 616 / 660 / 566 / 520 / 555 us). Measured against packing, the hop on packed fields and
// unpacking: 24^3x48 328 -> 185 us, 4^3x8 15.0 -> 11.6 us. Bound by the traffic between L2 and memory
// (2.0 kB per site at 6.9 TB/s against 960 B that it cannot do without): an XCD has 16,384 sites in
// flight, 12 MB of data through a 4 MB L2, so the z and t neighbours miss it.
#include "wd_hop.hpp"

namespace wd {

constexpr int AP_W = 64;        // sites per block
constexpr int AP_S = 13;        // 16-byte pieces per site in LDS (12 and a pad)

// the 64 sites from `base`: piece j of lane l is number 64 j + l of the run
__device__ __forceinline__ void run_load(const d2v* src, long base, long npiece, int lane, int dep, d2v r[12])
{
#pragma unroll
    for (int j = 0; j < 12; j++) {
        const long e = base * 12 + j * AP_W + lane + dep;
        r[j] = e < npiece ? gld<d2v>(src, e) : d2v{0.0, 0.0};
    }
}
__device__ __forceinline__ void run_put(d2v* buf, int lane, const d2v r[12])
{
    int s = lane / 12, c = lane % 12;
#pragma unroll
    for (int j = 0; j < 12; j++) {
        buf[s * AP_S + c] = r[j];
        s += 5;
        c += 4;
        if (c >= 12) {
            c -= 12;
            s += 1;
        }
    }
}

// one direction: the neighbour's spinor from the run starting at `base` (or memory), projection, link,
// accumulation as in hop_dir
template <int MU, int D, bool DAG>
__device__ __forceinline__ void apply_dir(const Geo& g, const d2v* __restrict__ src, const d2v* buf, long n, long base,
                                          int x, int y, int z, int t, const void* lk, const void* lk_nb, long lcs,
                                          cx<double> acc[12], int& dep)
{
    using T = double;
    const int step = MU == 0 ? 1 : MU == 1 ? g.X : MU == 2 ? g.X * g.Y : g.X * g.Y * g.Z;
    const int L = MU == 0 ? g.X : MU == 1 ? g.Y : MU == 2 ? g.Z : g.T;
    const int c = MU == 0 ? x : MU == 1 ? y : MU == 2 ? z : t;
    const long nb = D == 0 ? (c + 1 == L ? n - (long)step * (L - 1) : n + step)
                           : (c == 0 ? n + (long)step * (L - 1) : n - step);
    cx<T> W[9];
    if constexpr (D == 0) {
        load_link<L64_18, T, false>(lk, lcs, MU, (n >> 1) + dep, W);
    } else {
        cx<T> F[9];
        load_link<L64_18, T, false>(lk_nb, lcs, MU, (nb >> 1) + dep, F);
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) W[a * 3 + b] = cconj(F[b * 3 + a]);
    }
    cx<T> psi[12];
    const long k = nb - base;
    if (k >= 0 && k < AP_W) {
#pragma unroll
        for (int j = 0; j < 12; j++) {
            const d2v q = buf[(int)k * AP_S + j];
            psi[j] = mk<T>(q[0], q[1]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 12; j++) {
            const d2v q = gld<d2v>(src, nb * 12 + j);
            psi[j] = mk<T>(q[0], q[1]);
        }
    }
    constexpr bool minus = (D == 0) != DAG;  // projector 1 - gamma
    constexpr int E = Proj<MU>::E + (minus ? 0 : 2);
    constexpr int F = Proj<MU>::F + (minus ? 0 : 2);
    constexpr int I1 = Proj<MU>::I1, I2 = Proj<MU>::I2;
    cx<T> h1[3], h2[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        h1[a] = psi[a * 4 + 3] + mul_ik<-E>(psi[a * 4 + I1]);
        h2[a] = psi[a * 4 + 2] + mul_ik<-F>(psi[a * 4 + I2]);
    }
    const bool flip = MU == 3 && g.anti && (D == 0 ? t == g.T - 1 : t == 0);
#pragma unroll
    for (int a = 0; a < 3; a++) {
        cx<T> g1 = row_dot(W, a, h1), g2 = row_dot(W, a, h2);
        if (MU == 3 && flip) {
            g1 = -g1;
            g2 = -g2;
        }
        acc[a * 4 + 3] = acc[a * 4 + 3] + g1;
        acc[a * 4 + 2] = acc[a * 4 + 2] + g2;
        acc[a * 4 + I1] = acc[a * 4 + I1] + mul_ik<E>(g1);
        acc[a * 4 + I2] = acc[a * 4 + I2] + mul_ik<F>(g2);
    }
    order_after(acc, dep);
}

// first site of the run of neighbours of site n0's wave in direction (MU, D)
template <int MU, int D>
__device__ __forceinline__ long run_base(const Geo& g, long n0, int x, int y, int z, int t)
{
    // lane 0's coordinates
    const int c = __builtin_amdgcn_readfirstlane(MU == 1 ? y : MU == 2 ? z : t);
    const int step = MU == 1 ? g.X : MU == 2 ? g.X * g.Y : g.X * g.Y * g.Z;
    const int L = MU == 1 ? g.Y : MU == 2 ? g.Z : g.T;
    return D == 0 ? (c + 1 == L ? n0 - (long)step * (L - 1) : n0 + step) : (c == 0 ? n0 + (long)step * (L - 1) : n0 - step);
}

template <bool DAG>
__global__ __launch_bounds__(AP_W) void k_apply(double2* __restrict__ dst, const double2* __restrict__ src_, Geo g,
                                                const void* __restrict__ lk_even, const void* __restrict__ lk_odd,
                                                long lcs, double c0, int tb, int bps)
{
    __shared__ d2v run[AP_W * AP_S];
    const d2v* src = (const d2v*)src_;
    const long V = 2L * g.Vh, npiece = V * 12;
    const int lane = threadIdx.x;
    int blk = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    if (tb > 0) {  // t fastest within groups of tb blocks of a t-slice (as in tiled_block)
        const int per = tb * g.T, grp = blk / per, q = blk - grp * per;
        const int first = grp * tb, size = bps - first < tb ? bps - first : tb;
        const int tt = q / size;
        blk = first + (q - tt * size) + bps * tt;
    }
    const long n0 = (long)blk * AP_W;
    const bool ok = n0 + lane < V;
    const long n = ok ? n0 + lane : V - 1;  // lanes past the end repeat the last site, without storing it
    unsigned u = (unsigned)n;
    const int x = (int)(u % (unsigned)g.X);
    u /= (unsigned)g.X;
    const int y = (int)(u % (unsigned)g.Y);
    u /= (unsigned)g.Y;
    const int z = (int)(u % (unsigned)g.Z), t = (int)(u / (unsigned)g.Z);
    const bool odd = ((x + y + z + t) & 1) != 0;
    const void* lk = odd ? lk_odd : lk_even;
    const void* lk_nb = odd ? lk_even : lk_odd;
    cx<double> acc[12];
#pragma unroll
    for (int k = 0; k < 12; k++) acc[k] = mk<double>(0.0, 0.0);
    int dep = 0;
    d2v r[12];
    run_load(src, n0, npiece, lane, dep, r);
    run_put(run, lane, r);
    long base = run_base<1, 0>(g, n0, x, y, z, t);
    run_load(src, base, npiece, lane, dep, r);
    __syncthreads();
    apply_dir<0, 0, DAG>(g, src, run, n, n0, x, y, z, t, lk, lk_nb, lcs, acc, dep);
    apply_dir<0, 1, DAG>(g, src, run, n, n0, x, y, z, t, lk, lk_nb, lcs, acc, dep);
    __syncthreads();
#define AP_STEP(MU_, D_, MUN_, DN_)                                                                                \
    {                                                                                                              \
        const long cur = base;                                                                                     \
        run_put(run, lane, r);                                                                                     \
        base = run_base<MUN_, DN_>(g, n0, x, y, z, t);                                                             \
        run_load(src, base, npiece, lane, dep, r);                                                                 \
        __syncthreads();                                                                                           \
        apply_dir<MU_, D_, DAG>(g, src, run, n, cur, x, y, z, t, lk, lk_nb, lcs, acc, dep);                        \
        __syncthreads();                                                                                           \
    }
    AP_STEP(1, 0, 1, 1)
    AP_STEP(1, 1, 2, 0)
    AP_STEP(2, 0, 2, 1)
    AP_STEP(2, 1, 3, 0)
    AP_STEP(3, 0, 3, 1)
#undef AP_STEP
    run_put(run, lane, r);
    run_load(src, n0, npiece, lane, dep, r);  // the own spinors again (from L2): c0 psi
    __syncthreads();
    apply_dir<3, 1, DAG>(g, src, run, n, base, x, y, z, t, lk, lk_nb, lcs, acc, dep);
    __syncthreads();
    run_put(run, lane, r);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const d2v q = run[lane * AP_S + k];
        const cx<double> v = -0.5 * acc[k], o = v + c0 * mk<double>(q[0], q[1]);
        run[lane * AP_S + k] = d2v{o.re, o.im};
    }
    __syncthreads();
    int s = lane / 12, c = lane % 12;
#pragma unroll
    for (int j = 0; j < 12; j++) {
        const long e = n0 * 12 + j * AP_W + lane;
        if (e < npiece) gst<d2v, true>(dst, e, run[s * AP_S + c]);
        s += 5;
        c += 4;
        if (c >= 12) {
            c -= 12;
            s += 1;
        }
    }
}

hipError_t launch_apply(bool dag, double* dst, const double* src, const Geo& g, const void* lk_even, const void* lk_odd,
                        long lcs, double c0, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    const long V = 2L * g.Vh;
    const int slice = g.X * g.Y * g.Z;
    const int bps = slice / AP_W, tb = slice % AP_W == 0 ? 64 : 0;
    const dim3 grid = grid1((V + AP_W - 1) / AP_W);
    if (dag) hipExtLaunchKernelGGL((k_apply<true>), grid, dim3(AP_W), 0, s, ev0, ev1, 0, (double2*)dst,
                                   (const double2*)src, g, lk_even, lk_odd, lcs, c0, tb, bps);
    else hipExtLaunchKernelGGL((k_apply<false>), grid, dim3(AP_W), 0, s, ev0, ev1, 0, (double2*)dst,
                               (const double2*)src, g, lk_even, lk_odd, lcs, c0, tb, bps);
    return hipGetLastError();
}

} // namespace wd
