// wd_apply / wd_apply_dag / wd_apply_noalloc: M(kappa) (Sec. 2, eq. 3 and 4) in FP64 straight from and
// to the caller's canonical fields, both parities in one launch, no packed copies.
//
// One wavefront (one block) per 64 consecutive canonical sites of a time slice, and of the next slice where
// a block does two. A site's spinor is 192 contiguous bytes, so lanes that load their own or their
// neighbour's spinor would touch 64 cache lines per instruction; instead the wave has each of the runs of
// 64 sites that its stencil needs (its own, which also serves x +- 1, the y and z neighbours of its first
// site and the next slice's) loaded straight into LDS, 64 bytes of a site at a time. Lanes whose neighbour
// is not in the run (periodic wraps inside it) load it from memory. Two buffers: a run and its link
// arrive while the direction before is computed, without passing through registers. The backward time
// hop is formed a slice early, from the link and the spinors that are there then. The output goes back
// through LDS the same way.
//
// Links: the 18-real internal format, forward slots only (the backward link of a site is its
// neighbour's forward one, which the wave next to it uses as well). Lanes 2 i and 2 i + 1 are the two
// sites of checkerboard index i, one of each parity, so a wave reads 512 contiguous bytes of either
// parity's array per piece.
//
// Measured (start: packing, the hop on packed fields and unpacking / one buffer filled through registers,
// every slice by itself / this): 4^3x8 15.0 / 11.7 / 8.9 us, 16^3x32 - / 37.7 / 30.9, 24^3x48 328 / 184 / 178,
// 32^3x64 - / 523 / 518. Small lattices: a chain of one round trip to memory per direction. Large ones:
// the vector L1 is busy throughout and waits for lines from L2 in 60 % of its cycles (2.35 kB a site, 0.84
// to 1.8 kB of them from memory); LDS holds six waves a CU.
#include "wd_hop.hpp"

namespace wd {

constexpr int AP_W = 64;  // sites per block
typedef __attribute__((address_space(3))) d2v lds_d2v;

// A run of 64 sites in LDS, filled by twelve direct global -> LDS loads (lane l's 16 bytes go to the load's
// base + 16 l). Load j takes four pieces of each of 16 sites: lanes 4 q .. 4 q + 3 read 64 contiguous
// bytes of site 16 (j / 3) + q, in an order turned by q / 4, with which lanes that read the same piece of
// consecutive sites later meet no bank conflict.
__device__ __forceinline__ int run_piece(int lane) { return 12 * (lane >> 2) + ((lane + (lane >> 4)) & 3); }
__device__ __forceinline__ void fetch16(const d2v* g, lds_d2v* l)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
__device__ __forceinline__ void run_fetch(lds_d2v* buf, const d2v* src, long base, long npiece, int lane)
{
    // past the end of the field: its last piece again (no branch, so that the compiler can count the loads)
    const long left = npiece - base * 12 - 1;
    const unsigned lim = left < 767 ? (unsigned)left : 767u, e = (unsigned)run_piece(lane);
    const d2v* p = src + base * 12;
#pragma unroll
    for (int j = 0; j < 12; j++) {
        const unsigned k = e + 192 * (j / 3) + 4 * (j % 3);
        fetch16(p + (k < lim ? k : lim), buf + 64 * j);
    }
}
// where piece m (0..3) of site k's first four is; the next four are 64 further
__device__ __forceinline__ int run_slot(int k, int m) { return 192 * (k >> 4) + 4 * (k & 15) + ((m - (k >> 2)) & 3); }
__device__ __forceinline__ void run_get(const lds_d2v* buf, int k, cx<double> psi[12])
{
#pragma unroll
    for (int m = 0; m < 4; m++) {
        const int i = run_slot(k, m);
#pragma unroll
        for (int h = 0; h < 3; h++) {
            const d2v q = buf[i + 64 * h];
            psi[4 * h + m] = mk<double>(q[0], q[1]);
        }
    }
}
// every load of the wave has arrived, in registers and in LDS
__device__ __forceinline__ void run_wait()
{
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

struct RawLink {
    d2v q[9];
};
__device__ __forceinline__ RawLink raw_link(const void* lk, long lcs, int mu, long i)
{
    RawLink l;
#pragma unroll
    for (int j = 0; j < 9; j++) l.q[j] = gld<d2v>(lk, chunk_at(72, lcs, i, mu * 9 + j));
    return l;
}
__device__ __forceinline__ void order_after_link(const RawLink& l, int& dep)
{
#pragma unroll
    for (int j = 0; j < 9; j++) asm volatile("" ::"v"(l.q[j]));
    asm volatile("" : "+v"(dep));
}
template <bool CONJ>
__device__ __forceinline__ void link_of(const RawLink& l, cx<double> W[9])
{
#pragma unroll
    for (int a = 0; a < 3; a++)
#pragma unroll
        for (int b = 0; b < 3; b++) {
            const d2v q = l.q[CONJ ? b * 3 + a : a * 3 + b];
            W[a * 3 + b] = mk<double>(q[0], CONJ ? -q[1] : q[1]);
        }
}

// g1, g2 = W (the two projected spinors of psi) in direction (MU, D)
template <int MU, int D, bool DAG>
__device__ __forceinline__ void half_hop(const cx<double> psi[12], const cx<double> W[9], bool flip, cx<double> g1[3],
                                         cx<double> g2[3])
{
    constexpr bool minus = (D == 0) != DAG;  // projector 1 - gamma
    constexpr int E = Proj<MU>::E + (minus ? 0 : 2);
    constexpr int F = Proj<MU>::F + (minus ? 0 : 2);
    constexpr int I1 = Proj<MU>::I1, I2 = Proj<MU>::I2;
    cx<double> h1[3], h2[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        h1[a] = psi[a * 4 + 3] + mul_ik<-E>(psi[a * 4 + I1]);
        h2[a] = psi[a * 4 + 2] + mul_ik<-F>(psi[a * 4 + I2]);
    }
#pragma unroll
    for (int a = 0; a < 3; a++) {
        g1[a] = row_dot(W, a, h1);
        g2[a] = row_dot(W, a, h2);
        if (MU == 3 && flip) {
            g1[a] = -g1[a];
            g2[a] = -g2[a];
        }
    }
}
template <int MU, int D, bool DAG>
__device__ __forceinline__ void add_half(const cx<double> g1[3], const cx<double> g2[3], cx<double> acc[12])
{
    constexpr bool minus = (D == 0) != DAG;
    constexpr int E = Proj<MU>::E + (minus ? 0 : 2);
    constexpr int F = Proj<MU>::F + (minus ? 0 : 2);
    constexpr int I1 = Proj<MU>::I1, I2 = Proj<MU>::I2;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        acc[a * 4 + 3] = acc[a * 4 + 3] + g1[a];
        acc[a * 4 + 2] = acc[a * 4 + 2] + g2[a];
        acc[a * 4 + I1] = acc[a * 4 + I1] + mul_ik<E>(g1[a]);
        acc[a * 4 + I2] = acc[a * 4 + I2] + mul_ik<F>(g2[a]);
    }
}
// the neighbour of site n in direction (MU, D)
template <int MU, int D>
__device__ __forceinline__ long neighbour(const Geo& g, long n, int x, int y, int z, int t)
{
    const int step = MU == 0 ? 1 : MU == 1 ? g.X : MU == 2 ? g.X * g.Y : g.X * g.Y * g.Z;
    const int L = MU == 0 ? g.X : MU == 1 ? g.Y : MU == 2 ? g.Z : g.T;
    const int c = MU == 0 ? x : MU == 1 ? y : MU == 2 ? z : t;
    return D == 0 ? (c + 1 == L ? n - (long)step * (L - 1) : n + step) : (c == 0 ? n + (long)step * (L - 1) : n - step);
}
// its link: the forward one of the site or of its backward neighbour
template <int MU, int D>
__device__ __forceinline__ RawLink dir_link(const Geo& g, long n, int x, int y, int z, int t, const void* lk,
                                            const void* lk_nb, long lcs)
{
    if constexpr (D == 0) return raw_link(lk, lcs, MU, n >> 1);
    else return raw_link(lk_nb, lcs, MU, neighbour<MU, D>(g, n, x, y, z, t) >> 1);
}

// the neighbour's spinor from the run starting at `base`, or from memory
template <int MU, int D>
__device__ __forceinline__ void dir_spinor(const Geo& g, const d2v* __restrict__ src, const lds_d2v* buf, long n, long base,
                                           int x, int y, int z, int t, cx<double> psi[12])
{
    const long nb = neighbour<MU, D>(g, n, x, y, z, t), k = nb - base;
    if (k >= 0 && k < AP_W) {
        run_get(buf, (int)k, psi);
    } else {
#pragma unroll
        for (int j = 0; j < 12; j++) {
            const d2v q = gld<d2v>(src, nb * 12 + j);
            psi[j] = mk<double>(q[0], q[1]);
        }
        int dep = 0;
        order_after(psi, dep);  // these loads end here, not behind the ones that follow
    }
    asm volatile("" ::: "memory");
}
// projection, link, accumulation as in hop_dir
template <int MU, int D, bool DAG>
__device__ __forceinline__ void dir_add(const Geo& g, int t, const cx<double> psi[12], const RawLink& link,
                                        cx<double> acc[12], int& dep)
{
    cx<double> W[9], g1[3], g2[3];
    link_of<D == 1>(link, W);
    half_hop<MU, D, DAG>(psi, W, MU == 3 && g.anti && (D == 0 ? t == g.T - 1 : t == 0), g1, g2);
    add_half<MU, D, DAG>(g1, g2, acc);
    order_after(acc, dep);
}

// first site of the run of neighbours of the wave's run n0 in direction (MU, D), MU = 1 or 2
template <int MU, int D>
__device__ __forceinline__ long run_base(const Geo& g, long n0, int y, int z)
{
    // lane 0's coordinates
    const int c = __builtin_amdgcn_readfirstlane(MU == 1 ? y : z);
    const int step = MU == 1 ? g.X : g.X * g.Y;
    const int L = MU == 1 ? g.Y : g.Z;
    return D == 0 ? (c + 1 == L ? n0 - (long)step * (L - 1) : n0 + step) : (c == 0 ? n0 + (long)step * (L - 1) : n0 - step);
}

__device__ __forceinline__ void slice_coords(const Geo& g, int sl, int& x, int& y, int& z)
{
    const unsigned u = (unsigned)sl / (unsigned)g.X;
    x = sl - (int)u * g.X;
    z = (int)(u / (unsigned)g.Y);
    y = (int)u - z * g.Y;
}

// What a block carries from one time slice to the next
struct ApplyState {
    cx<double> b1[3], b2[3];  // the backward time hop of the coming slice
};

// One time slice: own holds its spinors, first the link of x+; both are the other's at the end (oth the
// next slice's spinors, second its link of x+).
template <bool DAG>
__device__ __forceinline__ void apply_slice(double2* __restrict__ dst, const d2v* src, const Geo& g, const void* lk_even,
                                            const void* lk_odd, long lcs, double c0, int slice, int s0, int lane0, int sl0,
                                            int t, bool more, lds_d2v* own, lds_d2v* oth, RawLink& first,
                                            RawLink& second, ApplyState& st)
{
    const long npiece = 24L * g.Vh;
    // opaque copies: what follows from them is formed again in every slice instead of being kept
    int lane = lane0, sl = sl0, dep = 0;
    asm volatile("" : "+v"(lane), "+v"(sl));
    int x, y, z;
    slice_coords(g, sl, x, y, z);
    const long n0 = (long)t * slice + s0, n = (long)t * slice + sl;
    const bool odd = ((x + y + z + t) & 1) != 0;
    const void* lk = odd ? lk_odd : lk_even;
    const void* lk_nb = odd ? lk_even : lk_odd;
    cx<double> acc[12];
#pragma unroll
    for (int k = 0; k < 12; k++) acc[k] = mk<double>(0.0, 0.0);
    // Loads run one direction ahead of the arithmetic: a direction's spinors go from LDS to registers, then
    // the next one's run and link are asked for, then this one is computed. (In this order because the
    // compiler has an LDS read wait for all loads into LDS.)
    cx<double> psi[12];
    dir_spinor<0, 0>(g, src, own, n, n0, x, y, z, t, psi);
    second = dir_link<0, 1>(g, n, x, y, z, t, lk, lk_nb, lcs);
    asm volatile("" ::: "memory");
    dir_add<0, 0, DAG>(g, t, psi, first, acc, dep);
    long base = run_base<1, 0>(g, n0, y, z);
    dir_spinor<0, 1>(g, src, own, n + dep, n0, x, y, z, t, psi);
    order_after_link(second, dep);  // it has arrived, before more is asked for
    first = dir_link<1, 0>(g, n, x, y, z, t, lk, lk_nb, lcs);
    run_fetch(oth, src, base, npiece, lane);
    asm volatile("" ::: "memory");
    dir_add<0, 1, DAG>(g, t, psi, second, acc, dep);
    run_wait();
#define AP_STEP(MU_, D_, HAVE_, MUN_, DN_, NEED_, BUF_, NEXT_, BASE_)                                              \
    dir_spinor<MU_, D_>(g, src, BUF_, n + dep, base, x, y, z, t, psi);                                             \
    NEED_ = dir_link<MUN_, DN_>(g, n, x, y, z, t, lk, lk_nb, lcs);                                                 \
    base = BASE_;                                                                                                  \
    run_fetch(NEXT_, src, base, npiece, lane);                                                                     \
    asm volatile("" ::: "memory");                                                                                 \
    dir_add<MU_, D_, DAG>(g, t, psi, HAVE_, acc, dep);                                                             \
    run_wait();
    AP_STEP(1, 0, first, 1, 1, second, oth, own, (run_base<1, 1>(g, n0, y, z)))
    AP_STEP(1, 1, second, 2, 0, first, own, oth, (run_base<2, 0>(g, n0, y, z)))
    AP_STEP(2, 0, first, 2, 1, second, oth, own, (run_base<2, 1>(g, n0, y, z)))
    AP_STEP(2, 1, second, 3, 0, first, own, oth, (long)(t + 1 == g.T ? 0 : t + 1) * slice + s0)
#undef AP_STEP
    dir_spinor<3, 0>(g, src, oth, n + dep, base, x, y, z, t, psi);
    run_fetch(own, src, n0, npiece, lane);  // the own spinors again (from L2)
    asm volatile("" ::: "memory");
    dir_add<3, 0, DAG>(g, t, psi, first, acc, dep);
    add_half<3, 1, DAG>(st.b1, st.b2, acc);
    run_wait();
    run_get(own, sl - s0, psi);
    if (more) second = dir_link<0, 0>(g, n + slice + dep, x, y, z, t + 1, lk_nb, lk, lcs);
    asm volatile("" ::: "memory");
    {
        cx<double> W[9];
        if (more) {
            link_of<true>(first, W);
            half_hop<3, 1, DAG>(psi, W, false, st.b1, st.b2);
        }
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const cx<double> v = -0.5 * acc[k];
            acc[k] = v + c0 * psi[k];
        }
    }
    __syncthreads();
    if (s0 + lane < slice) {
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const int i = run_slot(lane, m);
#pragma unroll
            for (int h = 0; h < 3; h++) own[i + 64 * h] = d2v{acc[4 * h + m].re, acc[4 * h + m].im};
        }
    }
    __syncthreads();
    const long e = n0 * 12 + run_piece(lane);
#pragma unroll
    for (int j = 0; j < 12; j++)
        if (s0 + 16 * (j / 3) + (lane >> 2) < slice)
            gst<d2v, true>(dst, e + 192 * (j / 3) + 4 * (j % 3), own[64 * j + lane]);
    __syncthreads();
}

// nt: time slices per block; ncol: columns of 64 sites per time slice; tb: columns per group. The blocks of a group
// run through the time ranges, so that what two neighbouring slices share is still in the XCD's L2.
template <bool DAG>
__global__ __launch_bounds__(AP_W, 2) void k_apply(double2* __restrict__ dst, const double2* __restrict__ src_, Geo g,
                                                   const void* __restrict__ lk_even, const void* __restrict__ lk_odd,
                                                   long lcs, double c0, int nt, int ncol, int tb)
{
    __shared__ d2v mema[AP_W * 12], memb[AP_W * 12];
    lds_d2v *bufa = (lds_d2v*)mema, *bufb = (lds_d2v*)memb;
    const d2v* src = (const d2v*)src_;
    const long npiece = 24L * g.Vh;
    const int slice = g.X * g.Y * g.Z, lane = threadIdx.x;
    const int blk = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int nch = (g.T + nt - 1) / nt, per = tb * nch, grp = blk / per, q = blk - grp * per;
    const int size = ncol - grp * tb < tb ? ncol - grp * tb : tb, ch = q / size;
    const int s0 = (grp * tb + q - ch * size) * AP_W;
    const int t0 = ch * nt, t1 = t0 + nt < g.T ? t0 + nt : g.T;
    const int sl = s0 + lane < slice ? s0 + lane : slice - 1;  // lanes past the end repeat the last site, without storing it
    ApplyState st;
    RawLink la, lb;
    {
        const int tm = t0 == 0 ? g.T - 1 : t0 - 1;
        int x, y, z;
        slice_coords(g, sl, x, y, z);
        const bool odd = ((x + y + z + t0) & 1) != 0;
        const long n = (long)t0 * slice + sl;
        run_fetch(bufb, src, (long)tm * slice + s0, npiece, lane);
        lb = raw_link(((x + y + z + tm) & 1) != 0 ? lk_odd : lk_even, lcs, 3, ((long)tm * slice + sl) >> 1);
        run_fetch(bufa, src, (long)t0 * slice + s0, npiece, lane);
        la = raw_link(odd ? lk_odd : lk_even, lcs, 0, n >> 1);
        run_wait();
        cx<double> W[9], psi[12];
        run_get(bufb, sl - s0, psi);
        link_of<true>(lb, W);
        half_hop<3, 1, DAG>(psi, W, g.anti && t0 == 0, st.b1, st.b2);
        __syncthreads();
    }
    for (int t = t0; t < t1; t += 2) {
        apply_slice<DAG>(dst, src, g, lk_even, lk_odd, lcs, c0, slice, s0, lane, sl, t, t + 1 < t1, bufa, bufb, la, lb, st);
        if (t + 1 < t1)
            apply_slice<DAG>(dst, src, g, lk_even, lk_odd, lcs, c0, slice, s0, lane, sl, t + 1, t + 2 < t1, bufb, bufa, lb, la, st);
    }
}

// Slices per block: one while all blocks find room on the chip at once (six to a CU), else two (one / two / four /
// eight: 8^3x16 8.6 / 13.5 / 24 / 46 us, 16^3x32 35.1 / 30.9 / 33.9 / 52, 20x14x18x30 38.9 / 38.9 / 40.6 / 65, 24^3x48
// 176 / 179 / 179 / 182, 32^3x64 529 / 518 / 540 / 556).
constexpr long AP_RESIDENT = 6 * 256;
// Columns per group of the block order, two slices per block (32 / 64 / 128 / all columns of a slice): 24^3x48
// 191 / 184 / 179 / 182 us, 32^3x64 598 / 526 / 518 / 580.
constexpr int AP_GROUP = 128;

hipError_t launch_apply(bool dag, double* dst, const double* src, const Geo& g, const void* lk_even, const void* lk_odd,
                        long lcs, double c0, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    const int slice = g.X * g.Y * g.Z, ncol = (slice + AP_W - 1) / AP_W;
    const int nt = (long)ncol * g.T <= AP_RESIDENT ? 1 : 2, tb = AP_GROUP < ncol ? AP_GROUP : ncol;
    const dim3 grid = grid1((long)ncol * ((g.T + nt - 1) / nt));
    if (dag) hipExtLaunchKernelGGL((k_apply<true>), grid, dim3(AP_W), 0, s, ev0, ev1, 0, (double2*)dst,
                                   (const double2*)src, g, lk_even, lk_odd, lcs, c0, nt, ncol, tb);
    else hipExtLaunchKernelGGL((k_apply<false>), grid, dim3(AP_W), 0, s, ev0, ev1, 0, (double2*)dst,
                               (const double2*)src, g, lk_even, lk_odd, lcs, c0, nt, ncol, tb);
    return hipGetLastError();
}

} // namespace wd
