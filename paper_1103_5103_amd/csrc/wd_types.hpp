// Structures shared by the host driver and the kernels of libwdirac.
//
// Every kernel launch works on a list of jobs held in device memory. A job is one (system,
// parity) pair: the blocks of a launch are split over the jobs, so a single launch can advance
// many independent systems of different lattice sizes at once (batched solves), and a
// full-lattice operator is simply two jobs, one per output parity.
//
// Solver scalars live on the device (SysState), one record per system. Reductions are
// deterministic: every block of a kernel writes one partial sum, and a small follow-up kernel
// (one block per system) adds the partials in a fixed order and then updates the scalars
// ("finisher"). The kernel boundary orders the two, so no device-wide fence is needed inside
// the bandwidth-bound kernels. Kernels launched with a gate (a mask of statuses) skip the
// systems whose status is not in it: the iteration runs RUNNING systems only, so a whole chunk
// of iterations can be queued without host round trips, and the steps between chunks (reliable
// updates, restarts) run on the full job tables with the mask of the systems they concern.
#pragma once
#include "wd_device.hpp"

namespace wd {

enum SysStatus {
    ST_RUNNING = 0,
    ST_CONVERGED = 1,   // iterated residual below target: verify with an FP64 residual
    ST_RELIABLE = 2,    // reliable update due
    ST_BREAKDOWN = 3,
    ST_NAN = 4,
    ST_MAXIT = 5,
    ST_DONE = 6,        // finished (no kernel runs it): the FP64 residual met the target, or set by the host
    ST_SEL1 = 7,        // selected for a gated step: continue after a reliable update / finish by sweep
    ST_SEL2 = 8,        //   restart fresh / finish by hop
    ST_NOCONV = 9,      // finished: iteration cap
    ST_BROKEN = 10,     // finished: broke down again after its restarts
};
// Finishers of small launches are folded into the sweep that follows: every block of the sweep adds the
// partial sums and computes the scalars itself, block 0 stores them (FIN_NONE: no finisher launch).
// The sweep after a hop writes its own partial sums while it reads the hop's, so the two hops of an
// iteration use one set each. What the scalars follow from is never written by the same launch: the
// last sweep of an iteration changes delta, iter and maxrr and reads the copies that the first one left.
// The exception is the gate: block 0 may store a status other than RUNNING before another block looks
// at it. That block then returns at the gate instead of after its own sums, which gave the same status:
// a sweep of a system that stops writes nothing in either case.
constexpr int FIN_NONE = -1;
// Kernel gates are masks of the statuses allowed to run (0: no gating); GATE_RUN = the iteration.
constexpr int GATE_RUN = 1 << ST_RUNNING;
// updates of these go on with the iteration unless the target is met (the others only verify)
constexpr int GATE_GOES_ON = (1 << ST_RELIABLE) | (1 << ST_BREAKDOWN);
constexpr int GATE_STOPPED = (1 << ST_CONVERGED) | (1 << ST_RELIABLE) | (1 << ST_BREAKDOWN) | (1 << ST_MAXIT);

// Finisher kinds (what follows from the reduced sums)
enum Fin {
    FIN_STORE = 0,   // keep the sums in red[] for the host
    FIN_BETA = 1,    // beta = -delta / <rhat, A s>
    FIN_RESTART = 5, // new residual: delta = <rhat, r>, |r|^2, status RUNNING
    FIN_CGA = 6,     // CG: alpha = |r|^2 / <p, A p>
    FIN_UPDATE = 8,  // FP64 residual update: |r|^2, finished or which way to go on
    FIN_CHIALPHA = 9,  // chi, delta' and alpha from the second hop's sums (fused sweep OP_XRS)
    FIN_RR = 10,     // |r|^2 of the fused sweep, status (+ the iteration's scalars for the shifts)
    FIN_CGB = 7,     // CG: beta = |r_new|^2 / |r|^2, status     (+ the iteration's scalars for the shifts)
};

// ---------------------------------------------------------------- shifted systems
// The shifted systems of BiCGstab-M / CG-M are not touched by the iteration. It leaves its residuals
// (BiCGstab-M: also w) in separate buffers and its scalars in a list; every SHIFT_BLOCK iterations
// the shifted x and s (CG-M: p) are brought up to date in one pass (wd_shift.hip). Over a block of
// m iterations x^s and s^s are linear combinations of themselves and of r_0, w_0, r_1, ..., r_m.
constexpr int SHIFT_BLOCK = 8;               // iterations per update, at most
constexpr int SHIFT_NB = 2 * SHIFT_BLOCK + 1;  // vectors of a block: r_0, w_0, r_1, ..., r_m

// the scalars of one iteration (CG-M: alpha_n, beta_{n+1} in the real parts)
struct IterScal {
    double2 beta, chi, alpha;
    double rr;
};

struct ShiftScal {
    double sigma;
    double2 zeta_prev, zeta;
    double2 rho;
    int active;      // 1: updated, 0: frozen
    int conv_iter;   // iteration at which the shift was frozen
};

// one shifted system's part of a block update:
//   x <- x + cx[0] s + sum_k cx[1 + k] v_k,  s <- cs[0] s + sum_k cs[1 + k] v_k
struct ShiftCoef {
    void* x;
    void* s;
    int store_s;  // 0: the shift was frozen in this block, s is not needed any more
    int pad;
    double2 cx[SHIFT_NB + 1], cs[SHIFT_NB + 1];
};

// what the iteration hands to the block update, and the update's own state (device memory, one per
// solve)
struct ShiftBlock {
    IterScal it[SHIFT_BLOCK];  // the iterations since the last update
    int count;                 // how many
    int updates;               // updates so far (the first one starts from x = 0, s = r_0)
    int first;                 // this update is the first one
    int nrun;                  // shifted systems in this update (entries of coef), -1: no update
    unsigned mask;             // which block vectors the update reads
    int pad;
    double2 alpha_prev, beta_prev;  // the base scalars before the block (CG-M: alpha, beta)
    double target2;  // a shift is frozen once its |r|^2 is below
};

// What a system reports to the host, in host memory that the device writes (even-odd solves): the host
// watches it instead of copying the record and waiting for the stream. state holds the status, the
// number of FP64 updates and the iteration in one word, stored after rr.
struct SysReport {
    double rr;                 // |r|^2: of the iterated residual, of the FP64 one where an update ends the solve
    unsigned long long state;  // status << 56 | updates << 32 | iteration
};

struct SysState {
    int status;        // SysStatus
    int nrel;          // FP64 residual updates so far
    int restarts;      // after breakdowns
    int pad;
    SysReport* report; // NULL: none
    int iter;
    int maxit;
    int mixed;
    int dc;            // defect correction: the reliable-update threshold is relative to the
                       // residual at the start of the inner solve (maxrr is not raised)
    double2 delta, beta, chi, alpha;
    double2 delta_w;   // folded finishers: delta, iter and maxrr as they were when w was formed
    double maxrr_w;
    int iter_w, pad2;
    double rr;         // |r|^2 of the iterated residual
    double maxrr;      // max |r|^2 since the last reliable update
    double rr_true;    // |r|^2 of the last FP64 residual update
    int fresh;         // x_lo counts as zero (start, after an update) and is not read
    int t_zero;        // T = D_oe x_hi counts as zero (no start vector, no update yet) and is not read
    double target2;    // stop when rr <= target2
    double delta_rel2; // reliable update when rr < delta_rel2 * maxrr
    double cga, cgb;   // CG: alpha_n, beta_n
    double red[NRED];  // last reduced sums
    double* partials;  // [max blocks][NRED]
    double* partials2; // a second set, for the second hop of an iteration with folded finishers
    ShiftBlock* blk;   // multi-shift solves: where the iteration leaves its scalars (else NULL)
};

// one entry per system of a launch: which partial sums the finisher adds
struct FinJob {
    int sys;
    int rnblk;
};

struct HopJob {
    Geo g;
    int parity;  // output parity
    int sys;     // SysState index (reduction group and gate)
    int blk0;    // first block of this job in the launch
    int nblk;
    int rblk0;   // first block within the system's reduction group
    int rnblk;   // blocks in the reduction group
    SpinorRef in;        // input half field (the other parity)
    SpinorRef out;       // output half field
    SpinorRef x0, x1;    // epilogue terms (p == nullptr: absent)
    SpinorRef z;         // partner of <z, out>
    // residual update (wd_update.hip): x_lo in z; the second hop's low-precision fields r, rhat, s, A s
    SpinorRef u_r, u_rh, u_s, u_as;
    int keep;            // residual update: the FP64 residual is stored whatever follows
    int s_current;       // residual update: s is up to date (fused sweep OP_XRS)
    const void* links;   // the 8 links per site of this output parity
    const void* links_nb;  // full-lattice launches: those of the other parity (else NULL)
    long lcs;            // link chunk stride
    double c0, c1, c2;   // out = c0 x0 + c1 x1 + c2 * hop
    int tb;              // block order: 0 = site order; > 0 = t fastest within groups of tb consecutive
                         // blocks of a t-slice (which is a whole number of blocks then)
    int bps;             // blocks per t-slice when tb > 0
    // Jobs that read the same links (same gauge field and parity) may form an interleaved group
    // of ilv consecutive jobs with equal blk0: block blk0 + ilv * l + k runs block l of job
    // (first + k), so the systems' blocks for one range of sites run together on one XCD and the
    // links come from memory once and from L2 for the others.
    int ilv;             // jobs in the group (1: not interleaved)
    int ilv_pos;         // position of this job in its group
    int tg;              // links in temporal gauge: the time links are the unit matrix except
                         // those leaving the last time slice (not loaded, not multiplied)
    // rhs >= 2: the group is run by the multi-RHS hop instead (k_hop_mrhs): one thread per output
    // site applies the hop to all ilv (<= rhs) systems of the group, loading each link once; the
    // group then spans nblk blocks rather than ilv * nblk. Every job of a launch has the same mode.
    int rhs;
    int split;           // run by the hop for small launches (blocks of SPLIT_SITES sites)
    int p2;              // partial sums go to the system's second set
    int nc;              // spinors in the non-chiral basis (gamma_4 diagonal): time hops read and
                         // update two spin components (hop_t_nc)
};

// Roles of the fields of a sweep job
enum SweepRole { R_F0 = 0, R_F1, R_F2, R_F3, R_F4, R_F5, R_F6, R_F7, NROLE };

struct SweepJob {
    int sys;
    int n;       // sites
    int blk0;
    int nblk;
    int rblk0;
    int rnblk;
    int flags;   // op-specific
    int pnblk;   // folded finishers: partial sums that the hop before this sweep left
    double c[8]; // op-specific coefficients
    SpinorRef f[NROLE];
};

} // namespace wd
