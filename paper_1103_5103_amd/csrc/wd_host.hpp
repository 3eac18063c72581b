// Host-side internals of libwdirac: the gauge handle, workspace fields, job tables and the
// error/timing plumbing shared by the solver drivers and the C ABI.
#pragma once
#include <hip/hip_runtime.h>

#include <chrono>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "../../include/wdirac.h"
#include "wd_kernels.hpp"

namespace wd {

// ---------------------------------------------------------------- errors
struct Error {
    wd_status code;
    std::string msg;
};
void set_error(const std::string& msg);
#define WD_CHECK_HIP(call)                                                                                       \
    do {                                                                                                         \
        hipError_t e_ = (call);                                                                                  \
        if (e_ != hipSuccess)                                                                                    \
            throw ::wd::Error{WD_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_)};                    \
    } while (0)
#define WD_REQUIRE(cond, msg)                                                                                    \
    do {                                                                                                         \
        if (!(cond)) throw ::wd::Error{WD_ERR_ARG, msg};                                                         \
    } while (0)

// ---------------------------------------------------------------- device memory
// A device allocation. Those of a destroyed handle (retire) are kept for the next handle's of the same size,
// up to 1 GiB a process while the device has 8 GiB free, the oldest given back first and all of them when an
// allocation fails or trim_memory() is called: what is
// given back to the driver it wipes at some 25 GB/s, and a program that makes a handle for every step of a
// training loop waits for that in the long run (16^3x32 forward and backward
// 4.0 ms, 15.7 ms where memory has been through many hands; with the list 3.1 ms).
struct DevMem {
    void* p = nullptr;
    size_t bytes = 0;
    std::shared_ptr<DevMem> owner;  // set: this is a part of another allocation, which it keeps alive
    int dev = -1;
    bool retired = false;
    DevMem() = default;
    explicit DevMem(size_t n);
    DevMem(const std::shared_ptr<DevMem>& whole, size_t off, size_t n) : p((char*)whole->p + off), bytes(n), owner(whole) {}
    ~DevMem();
    // no work on device `cur` uses the allocation any more: keep it for another handle when it is destroyed
    void retire(int cur)
    {
        DevMem& m = owner ? *owner : *this;
        m.retired = m.dev == cur;
    }
    DevMem(const DevMem&) = delete;
    DevMem& operator=(const DevMem&) = delete;
};

// An internal spinor field: one half (one parity) or a full field (both halves).
struct Field {
    std::shared_ptr<DevMem> mem;
    int sf = SF64;
    int halves = 1;
    long stride = 0;  // sites per half
    char* base() const { return (char*)mem->p; }
    float* nrm() const { return sf == SF16 ? (float*)(base() + (size_t)16 * spinor_chunks(sf) * halves * stride) : nullptr; }
    long cs() const { return stride * halves; }
    // view of parity p (a full field) or of the single half
    SpinorRef half(int p) const
    {
        SpinorRef r;
        r.p = base() + (size_t)p * stride * 16 * (AOSOA ? spinor_chunks(sf) : 1);
        float* n = nrm();
        r.nrm = n ? n + (size_t)p * stride : nullptr;
        r.cs = cs();
        return r;
    }
    SpinorRef all() const { return SpinorRef{base(), nrm(), cs()}; }
    long nsites() const { return stride * halves; }
};
void trim_memory();  // gives back the allocations of destroyed handles and the rooms that no solve uses
size_t field_bytes(int sf, int halves, long stride);
size_t room_of(size_t bytes);  // rounded up to what a part of an allocation takes

// ---------------------------------------------------------------- timing
// TK_HOP_LO_RED + r: the low-precision hops with fused reduction r (RED_NONE .. RED_FULL), also
// counted in TK_HOP_LO
enum { TK_HOP_LO = 0, TK_HOP_F64 = 1, TK_SWEEP = 2, TK_FINISH = 3, TK_HOP_LO_RED = 4, NTK = 9 };
struct Timer {
    bool on = false;
    struct Rec { int cls; hipEvent_t a, b; double bytes; int slot; int njobs; int cls2; };
    std::vector<Rec> pending;
    std::vector<hipEvent_t> pool;
    // pending holds at most kRecords (flush() reads as many flags back); every record goes through push()
    static constexpr size_t kRecords = 1 << 16;
    int* dflags = nullptr;  // per pending launch: set by the kernel when it did work
    int* slot();            // the flag of the next record, which is pushed before any other
    void push(const Rec& r);
    double ms[NTK] = {};
    double bytes[NTK] = {};
    long launches[NTK] = {};
    hipEvent_t get();
    void flush();
};
Timer& timer();

// ---------------------------------------------------------------- job tables
// A launch's job list (and the list of systems its finisher reduces) in device memory. A table
// owns its device copy (upload), or several tables share one buffer and one copy (upload_tables).
struct JobTableBase {
    std::shared_ptr<DevMem> dev;
    size_t off = 0;  // byte offset of this table in dev
    size_t cap = 0;  // bytes reserved for this table at off
    long nblocks = 0;
    virtual ~JobTableBase() = default;
    virtual size_t prepare() = 0;          // finisher list, nblocks; returns the image size
    virtual void write(char* dst) const = 0;  // the image: jobs, then the finisher list
};

template <class J>
struct JobTable : JobTableBase {
    std::vector<J> host;
    std::vector<FinJob> fin;  // one entry per system, for the finisher kernel
    void upload(hipStream_t s);
    size_t prepare() override;
    void write(char* dst) const override;
    int n() const { return (int)host.size(); }
    const J* d() const { return (const J*)((const char*)dev->p + off); }
    const FinJob* fin_d() const { return (const FinJob*)((const char*)dev->p + off + fin_offset()); }
    size_t fin_offset() const { return (host.size() * sizeof(J) + 255) / 256 * 256; }
};

// Upload several non-empty tables with one host-to-device copy into mem (grown when too small;
// tables still holding the previous buffer keep it alive).
void upload_tables(hipStream_t s, std::shared_ptr<DevMem>& mem, const std::vector<JobTableBase*>& tables);

// ---------------------------------------------------------------- gauge handle
} // namespace wd

struct wd_gauge {
    wd::Geo geo;
    long V = 0;
    std::unique_ptr<wd::DevMem> links[wd::NLINKFMT];  // both output parities, [parity][8][chunks][stride]
    // Solvers work in temporal gauge when the links are SU(3) to rounding: sources are rotated by
    // g(n) on the way in, solutions by g(n)^dag on the way out, and the solver link formats are
    // built from the transformed links (links[] keeps the caller's gauge for wd_apply and the
    // gradient).
    bool tg = false;
    // Solvers work in the non-chiral spin basis (gamma_4 diagonal) when the handle was created with
    // that option: sources are rotated on the way in, solutions on the way out, and the hops take
    // the time direction in that basis (half-spinor neighbours). wd_apply, wd_apply_noalloc and the
    // gradient use the caller's basis.
    int nc = 0;
    std::unique_ptr<wd::DevMem> gmat;                   // g(n), canonical [V][3][3] complex128
    std::unique_ptr<wd::DevMem> fixed[wd::NLINKFMT];    // transformed links, same layouts
    const double* gm() const { return tg ? (const double*)gmat->p : nullptr; }
    const void* slk(int lf, int parity) const;          // links of format lf for the solvers
    void ensure_slinks(int lf, hipStream_t s);
    std::map<std::string, wd::Field> ws;              // cached workspace fields
    std::map<std::string, std::shared_ptr<wd::DevMem>> raw;
    std::map<std::string, std::shared_ptr<void>> graphs;  // captured iteration chunks by launch key
    hipStream_t stream = nullptr;
    double recon_err = 1.0;  // max |row2 - conj(row0 x row1)| over the links
    double u00_max = 1.0;    // max |u00|^2 over the links (the 8-real format needs it below 1)
    // FP64 operator format of the solvers: 12-real when the links are SU(3) to rounding, else 18-real
    int f64_links() const { return recon_err < 1e-12 ? wd::L64_12 : wd::L64_18; }
    const void* lk(int lf, int parity) const;
    long lcs() const { return geo.stride; }
    wd::Field& field(const std::string& key, int sf, int halves);
    // The missing ones of these fields in one allocation per group, zeroed: giving memory back takes
    // about 0.24 ms an allocation (of 25 MB or more), whatever its size. 16^3x32 forward and backward
    // with a handle of its own: 7.0 ms with an allocation per field, of which 3.3 ms for giving 16 of
    // them back; 4.0 ms so. An allocation lives as long as any of its fields, so a group holds fields that
    // change their format together: the FP64 ones that never do (0), or those of one system's iteration.
    // Fields whose format has changed are given back first. A group of one field is left to field(), as
    // are those that the device does not have room for in one piece.
    struct FieldSpec {
        std::string key;
        int sf, halves, group = 0;
    };
    void reserve(const std::vector<FieldSpec>& fields);
    void* rawbuf(const std::string& key, size_t bytes);
    // Memory that a solve is faster with but can do without (zeroed when made; NULL: the device has no
    // room). The handle keeps it for its next solve; when an allocation of the library fails, those
    // that no solve holds are given back, whichever handle keeps them.
    std::shared_ptr<wd::DevMem> room(const std::string& key, size_t bytes);
    ~wd_gauge();
    // the same for the link formats that a handle makes when it is created
    void reserve_links(std::initializer_list<int> fmts);
    std::unique_ptr<wd::DevMem> new_links(int lf);
    std::shared_ptr<wd::DevMem> link_room;  // set while the handle is made
    size_t link_used = 0;
    void ensure_links(int lf, hipStream_t s);
    void build_temporal_gauge(const double* U, hipStream_t s);  // U: the caller's canonical links
    size_t device_bytes() const;
    void retire();  // the device is idle and the handle about to be destroyed
};

namespace wd {

// pinned staging for small host<->device copies (one buffer: synchronise before reusing it)
void* pinned(size_t bytes);
// pinned ring for host-to-device copies: no synchronisation needed, since a region is only
// handed out again after the device has drained (the ring synchronises when it wraps)
char* stage_alloc(size_t bytes);

// Host memory for the reports of one solve's systems (at most kMaxReports), taken from a process-wide
// pool and given back when the solve ends. A solve ends with finish(): the stream drains, and an error of
// the kernels queued last (they write the solutions) is the solve's. The destructor drains it where an
// exception has ended the solve. The pool keeps at most kReportPool blocks, the rest is freed. Safe with
// several threads.
constexpr int kMaxReports = 1024;
constexpr int kReportPool = 16;
struct Reports {
    volatile SysReport* r = nullptr;
    hipStream_t st;
    bool drained = false;  // finish() has been called
    explicit Reports(hipStream_t s);
    ~Reports();
    void finish()
    {
        WD_CHECK_HIP(hipStreamSynchronize(st));
        drained = true;
    }
    Reports(const Reports&) = delete;
    Reports& operator=(const Reports&) = delete;
    struct View {
        int status, nrel, iter;
        double rr;
    };
    View get(int i) const;
    // wait until ok(view) holds for system i; throws if the stream ends or fails without it
    template <class F>
    View wait(int i, F&& ok) const
    {
        bool drained = false;
        std::chrono::steady_clock::time_point since;
        for (long n = 1;; n++) {
            const View v = get(i);
            if (ok(v)) return v;
            if (!drained) {
                drained = pause(n);
                since = std::chrono::steady_clock::now();
            } else if (std::chrono::steady_clock::now() - since > std::chrono::seconds(1)) {  // (a report may become visible after the stream's end does)
                throw Error{WD_ERR_HIP, "the stream ended without the report of system " + std::to_string(i)};
            }
        }
    }
    // a moment's wait, now and then a look at the stream; true: it had drained
    bool pause(long n) const;
};

// wd_apply_noalloc: a fixed device array per GPU (kNoallocScratchBytes) takes a copy of an input that
// overlaps the output (at most 33.5 MB). The largest lattice is a limit of the interface, whether or not
// a call needs the copy: what it refuses does not depend on how the operator is applied.
constexpr size_t kNoallocScratchBytes = (size_t)64 << 20;
constexpr long kNoallocMaxStride = 87296;  // sites per parity, rounded up to whole blocks
constexpr int kNoallocMaxDevices = 64;
static_assert((size_t)2 * kNoallocMaxStride * 192 <= kNoallocScratchBytes, "the copy of an input fits");
void apply_noalloc(wd_gauge* g, double kappa, double* out, const double* in, bool dag, hipStream_t s);

// do two device ranges of this many bytes share an address
inline bool ranges_overlap(const void* a, const void* b, size_t bytes)
{
    return (const char*)a < (const char*)b + bytes && (const char*)b < (const char*)a + bytes;
}

// launch helpers with optional timing
// out = M(kappa) in or M^dag in on canonical FP64 fields that do not overlap
void run_apply(wd_gauge* g, double kappa, double* out, const double* in, bool dag, hipStream_t s);
// stage / ntl: -1 the defaults (LDS staging as built; non-temporal link loads unless the launch's
// links are shared or small), else forced (0 off, 1 on)
void run_hop(int sf, int lf, bool dag, int red, int fin, const JobTable<HopJob>& t, SysState* sys, int gated,
             hipStream_t s, double bytes_per_site_total, int stage = -1, int ntl = -1);
// a hop of an FP64 residual update (launch_update), gated on the stopped statuses; hop 2 is followed by
// FIN_UPDATE
void run_update(int hop, int sf, int lf, const JobTable<HopJob>& t, SysState* sys, hipStream_t s, double bytes_total);
// fold: the sweep does the finisher of the reduction before it and leaves its own to the next sweep
void run_sweep(int op, int sfl, const JobTable<SweepJob>& t, SysState* sys, int gated, hipStream_t s,
               double bytes_total, bool fold = false);
// the block update of the shifted systems (launch_shift_update), timed as a sweep
void run_shift_update(int nb, const ShiftVectors& v, long n, const ShiftBlock* blk, const ShiftCoef* coef,
                      hipStream_t s, double bytes_total);

int spinor_fmt_of(wd_prec p);
int link_fmt_of(wd_prec p, int recon);

} // namespace wd
