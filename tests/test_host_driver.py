"""CPU checks of the library's host code against a stand-in for the device (no GPU).

tests/host_driver_probe.cpp replaces the HIP runtime and the kernels: device memory with a capacity and
range checks, a queue in place of the stream, and scripted ends of iterations and FP64 updates. What is
checked is what the host does with them: which steps it queues, what it waits for and returns, and
what memory it holds. The fields hold no numbers.
"""
import concurrent.futures as cf
import ctypes
import os
import shutil
import subprocess

import pytest

import paper_1103_5103_amd as wd
from paper_1103_5103_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1103_5103_amd", "csrc")
HIP_ERROR, OOM, NOCONV, NAN, BREAKDOWN = 2, 3, 4, 6, 5


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("host_driver")
    src = [os.path.join(CSRC, f) for f in ("wd_runtime.cpp", "wd_solve.cpp", "wd_api.cpp")]
    src.append(os.path.join(ROOT, "tests", "host_driver_probe.cpp"))
    objs = [str(d / (os.path.basename(s) + ".o")) for s in src]

    def compile_one(s, o):
        subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-fPIC", "-I", CSRC, "-c", s, "-o", o],
                       check=True, capture_output=True)

    with cf.ThreadPoolExecutor(4) as ex:
        list(ex.map(compile_one, src, objs))
    so = str(d / "libhost.so")
    # -Bsymbolic: the stand-in's HIP calls, whatever else the process has loaded
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-o", so, *objs], check=True, capture_output=True)
    L = ctypes.CDLL(so)
    for f in ("fake_live", "fake_peak", "wd_gauge_device_bytes"):
        getattr(L, f).restype = ctypes.c_size_t
    with pytest.MonkeyPatch.context() as m:
        m.setenv("WD_TUNE_CACHE", str(d / "tune.txt"))
        yield L


class Host:
    """A handle of the stand-in library on a lattice, and calls on it (every device field at one address)."""

    def __init__(self, lib, dims, hint=None):
        self.lib, self.h = lib, ctypes.c_void_p()
        self.x = ctypes.c_void_p(1 << 40)  # never touched: the kernels compute nothing
        geom = _lib.Geom((ctypes.c_int * 4)(*dims), 1)
        assert lib.wd_gauge_create(ctypes.byref(self.h), ctypes.byref(geom), self.x,
                                   ctypes.byref(hint) if hint is not None else None, None) == 0

    def params(self, **kw):
        return params(self.lib, **kw)

    def solve(self, p, kappa=0.12):
        st = wd.SolverStats()
        code = self.lib.bicgstab_solve(self.h, ctypes.c_double(kappa), self.x, self.x, ctypes.byref(p), ctypes.byref(st), None)
        return code, [st]

    def batch(self, p, n):
        arr = (_lib.System * n)()
        for s in arr:
            s.gauge, s.kappa, s.b, s.x = self.h, 0.12, self.x, self.x
        st = (wd.SolverStats * n)()
        return self.lib.wd_batch_solve(n, arr, ctypes.byref(p), st, None), list(st)

    def masses(self, p, n, method, normal=False):
        v = (ctypes.c_double * n)(*[0.12 + 0.001 * i for i in range(n)])
        xs = (ctypes.c_void_p * n)(*[self.x.value] * n)
        st = (wd.SolverStats * n)()
        if normal:
            code = self.lib.wd_normal_solve(self.h, ctypes.c_double(0.12), n, v, xs, self.x, method, 1, ctypes.byref(p), st, None)
        else:
            code = self.lib.wd_multimass_solve(self.h, n, v, xs, self.x, method, 1, ctypes.byref(p), st, None)
        return code, list(st)

    def bytes(self):
        return self.lib.wd_gauge_device_bytes(self.h)

    def close(self):
        assert self.lib.wd_gauge_destroy(self.h) == 0


def params(lib, **kw):
    p = wd.SolverParams()
    lib.wd_params_default(ctypes.byref(p))
    for k, v in kw.items():
        assert hasattr(p, k)
        setattr(p, k, v)
    return p


def reset(lib, capacity=1 << 62, seed=1):
    lib.fake_reset(ctypes.c_size_t(capacity), seed)


def drop_spares(lib):
    """Allocations of closed handles go when an allocation fails."""
    reset(lib, capacity=0)
    h, geom = ctypes.c_void_p(), _lib.Geom((ctypes.c_int * 4)(4, 4, 4, 4), 1)
    assert lib.wd_gauge_create(ctypes.byref(h), ctypes.byref(geom), ctypes.c_void_p(1 << 40), None, None) == OOM
    reset(lib)


def script(lib, *p):
    lib.fake_script(*[ctypes.c_double(v) for v in p])


def last_error(lib):
    buf = ctypes.create_string_buffer(512)
    lib.wd_last_error(buf, 512)
    return buf.value.decode()


# ---------------------------------------------------------------- the schedule of the even-odd solves
SCRIPTS = {  # reliable, converged, verified, breakdown, nan
    "reliable": (0.3, 0.1, 1.0, 0.0, 0.0),
    "failed checks": (0.1, 0.3, 0.2, 0.0, 0.0),
    "everything": (0.2, 0.15, 0.4, 0.05, 0.02),
    "iteration cap": (0.2, 0.0, 0.0, 0.0, 0.0),
}


@pytest.mark.parametrize("dims,n", [((4, 4, 4, 4), 1), ((4, 4, 4, 4), 2), ((4, 4, 4, 4), 7), ((16, 16, 16, 16), 9)])
@pytest.mark.parametrize("kind", SCRIPTS)
@pytest.mark.parametrize("dc", [0, 1])
def test_systems_that_stop_at_different_times(lib, dims, n, kind, dc):
    """Whatever order the systems of a solve stop, go on, fail their check and restart in, the host
    neither loses count of one (it would wait for a report that never comes) nor gives up early.
    ((16, 16, 16, 16) x 9: above the folded finishers.)"""
    reset(lib)
    g = Host(lib, dims)
    for seed in range(8):
        reset(lib, seed=seed)
        script(lib, *SCRIPTS[kind])
        p = g.params(max_iter=30, mixed_mode=dc)
        code, st = g.batch(p, n) if n > 1 else g.solve(p)
        assert code != HIP_ERROR, (seed, last_error(lib))
        for s in st:
            assert 0 <= s.iters <= 30
            if kind == "iteration cap":
                assert (s.iters, s.status) == (30, NOCONV)
            elif kind == "reliable":
                assert s.status in (0, NOCONV) and s.reliable_updates > 0
        assert lib.fake_out_of_range() == 0
    g.close()


# ---------------------------------------------------------------- timing
def test_timing_of_more_launches_than_it_has_room_for(lib):
    """Every timed launch leaves a record; 65536 of them are read back at a time, whatever kind of
    launch the last one is."""
    reset(lib)
    g = Host(lib, (4, 4, 4, 4))
    script(lib, 0.0, 0.1, 1.0, 0.0, 0.0)
    out = ctypes.c_void_p(1 << 41)
    ms, n, by = ctypes.c_double(), ctypes.c_long(), ctypes.c_double()
    lib.wd_timing_reset()
    lib.wd_timing_enable(1)
    try:
        code, st = g.solve(g.params(max_iter=100))
        assert code == 0
        assert lib.wd_timing_get(1, ctypes.byref(ms), ctypes.byref(n), ctypes.byref(by)) == 0
        before = n.value
        for _ in range(70000):
            assert lib.wd_apply(g.h, ctypes.c_double(0.12), out, g.x, None) == 0
        assert lib.wd_timing_get(1, ctypes.byref(ms), ctypes.byref(n), ctypes.byref(by)) == 0
        assert n.value == before + 70000
        # a record at the last place of the buffer, and the finisher's behind it
        for k in range(65536 - 4, 65536 + 1):
            lib.wd_timing_reset()
            for _ in range(k):
                assert lib.wd_apply(g.h, ctypes.c_double(0.12), out, g.x, None) == 0
            assert g.solve(g.params(max_iter=100))[0] == 0
            assert lib.wd_timing_get(3, ctypes.byref(ms), ctypes.byref(n), ctypes.byref(by)) == 0
    finally:
        lib.wd_timing_enable(0)
    assert lib.fake_out_of_range() == 0
    g.close()


# ---------------------------------------------------------------- errors of the last kernels
@pytest.mark.parametrize("call", ["single", "batch", "sequential", "batched", "multishift"])
def test_a_failure_of_the_last_kernels_is_returned(lib, call):
    """The kernels that write the solutions are the last ones queued; when they fail, the solve that
    queued them says so."""
    reset(lib)
    g = Host(lib, (4, 4, 4, 4))
    script(lib, 0.1, 0.2, 1.0, 0.0, 0.0)
    p, f64 = g.params(max_iter=100), g.params(max_iter=100, mixed=0, eo=0)
    run = {"single": lambda: g.solve(p), "batch": lambda: g.batch(p, 3), "sequential": lambda: g.masses(p, 1, 0),
           "batched": lambda: g.masses(p, 3, 2), "multishift": lambda: g.masses(f64, 3, 1)}
    if call == "multishift":
        script(lib, 0.0, 1.0, 1.0, 0.0, 0.0)
    assert run[call]()[0] == 0
    lib.fake_fail_unpack()
    assert run[call]()[0] == HIP_ERROR
    reset(lib)
    g.close()


# ---------------------------------------------------------------- memory
F64, F32, F16 = 0, 1, 2  # wd_prec


def _spinors(g, f):
    return g.params(max_iter=100, mixed=0) if f == F64 else g.params(max_iter=100, spinor_store=f)


def _held(lib, dims, calls):
    """Device memory that a handle holds after each of these calls, and the handle's own count of it."""
    drop_spares(lib)
    script(lib, 0.1, 0.2, 1.0, 0.0, 0.0)
    base = lib.fake_live()
    g = Host(lib, dims, params(lib))
    out = []
    for f, n in calls:
        p = _spinors(g, f)
        assert (g.solve(p) if n == 1 else g.batch(p, n))[0] == 0
        out.append((lib.fake_live() - base, g.bytes()))
    g.close()
    assert lib.fake_live() == base
    return out


@pytest.mark.parametrize("seq", [(F32, F16), (F32, F16, F32), (F64, F32), (F64, F32, F64, F16), (F16, F64, F32, F16)])
def test_a_change_of_storage_gives_the_old_fields_back(lib, seq):
    """A handle that went through other formats holds what one holds that has only run the last."""
    dims = (4, 4, 4, 8)  # (allocations too small to be kept for the next handle)
    for n in (1, 2):
        _held(lib, dims, [(f, n) for f in seq])  # (the hop tuner's first run needs a buffer)
        got = _held(lib, dims, [(f, n) for f in seq])
        want = _held(lib, dims, [(seq[-1], n)])
        assert got[-1][0] == want[-1][0], (seq, n)
        assert all(live == count for live, count in got)


def test_a_change_of_storage_of_some_systems(lib):
    """The fields of one system of a batch are given back when it changes, though the others keep theirs."""
    dims = (4, 4, 4, 8)
    d = _held(lib, dims, [(F16, 1)])[0][0] - _held(lib, dims, [(F32, 1)])[0][0]
    got = _held(lib, dims, [(F32, 2), (F16, 1)])
    assert got[1][0] == got[0][0] + d


@pytest.mark.parametrize("seq", [(F32, F16, F32), (F64, F32, F64)])
def test_a_change_of_storage_where_memory_is_short(lib, seq):
    """The old fields are given back before the new ones are made: a device that has room for either set
    is enough."""
    dims = (4, 4, 4, 8)
    drop_spares(lib)
    script(lib, 0.1, 0.2, 1.0, 0.0, 0.0)
    base = lib.fake_live()
    g = Host(lib, dims, params(lib))
    limit = 0
    for f in set(seq):
        assert g.solve(_spinors(g, f))[0] == 0
        limit = max(limit, lib.fake_live())
    for f in seq:
        reset(lib, capacity=limit)
        script(lib, 0.1, 0.2, 1.0, 0.0, 0.0)
        assert g.solve(_spinors(g, f))[0] == 0, last_error(lib)
    g.close()
    assert lib.fake_live() == base


BLOCK_FIELDS = 15  # BiCGstab-M: what it holds beyond the fields that an update in every iteration needs


def _full_field(dims):
    v = dims[0] * dims[1] * dims[2] * dims[3]
    return 2 * ((v // 2 + 255) // 256 * 256) * 192


@pytest.mark.parametrize("other", ["more masses", "even-odd", "another handle", "normal"])
def test_vectors_kept_for_block_updates_give_way(lib, other):
    """The residuals that BiCGstab-M (CG-M) keeps for its block updates are given back when an
    allocation needs the room, whoever makes it: a call that fits without them is not refused because
    an earlier solve left them."""
    dims = (8, 8, 8, 8)
    drop_spares(lib)
    script(lib, 0.0, 0.2, 1.0, 0.0, 0.0)
    f64, eo = params(lib, max_iter=100, mixed=0, eo=0), params(lib, max_iter=100, mixed=0)
    g, g2 = Host(lib, dims, params(lib)), Host(lib, dims, params(lib))
    one = _full_field(dims)
    normal = other == "normal"
    calls = {"more masses": lambda: g.masses(f64, 6, 1), "even-odd": lambda: g.solve(eo), "another handle": lambda: g2.solve(eo),
             "normal": lambda: g.masses(f64, 6, 1)}
    before = lib.fake_live()
    assert g.masses(f64, 2, 1, normal=normal)[0] == 0
    kept = lib.fake_live()
    assert kept - before > (7 * one // 2 if normal else BLOCK_FIELDS * one)
    # room for the fields of the second call (BiCGstab-M of 6 masses without blocks: 8 more; even-odd FP64: 8),
    # less than the kept vectors take
    room = 0 if not normal else 20 * one
    for k in range(2):
        reset(lib, capacity=kept + room)
        script(lib, 0.0, 0.2, 1.0, 0.0, 0.0)
        assert calls[other]()[0] == 0, last_error(lib)
        # and the first call comes back, with shorter blocks if need be
        assert g.masses(f64, 2, 1, normal=normal)[0] == 0, last_error(lib)
    assert lib.fake_out_of_range() == 0
    g.close()
    g2.close()


def test_memory_of_closed_handles(lib):
    """Kept for the next handle up to 1 GiB, given back on request; not kept where the device is short."""
    dims = (16, 16, 16, 16)
    drop_spares(lib)
    script(lib, 0.1, 0.2, 1.0, 0.0, 0.0)
    base = lib.fake_live()

    def one():
        g = Host(lib, dims, params(lib))
        assert g.solve(params(lib, max_iter=100))[0] == 0
        g.close()

    one()
    kept = lib.fake_live()
    assert base < kept <= base + (1 << 30)
    one()
    assert lib.fake_live() == kept  # taken again
    assert lib.wd_trim_memory() == 0
    assert lib.fake_live() == base
    g = Host(lib, dims, params(lib))  # rooms of live handles
    f64 = params(lib, max_iter=100, mixed=0, eo=0)
    assert g.masses(f64, 2, 1)[0] == 0
    with_room = lib.fake_live()
    assert lib.wd_trim_memory() == 0
    assert lib.fake_live() == with_room - 14 * _full_field(dims)
    assert g.masses(f64, 2, 1)[0] == 0
    assert lib.fake_live() == with_room
    g.close()
    one()
    assert lib.fake_live() > base
    reset(lib, capacity=lib.fake_live() + (4 << 30))
    script(lib, 0.1, 0.2, 1.0, 0.0, 0.0)
    one()
    assert lib.fake_live() == base


@pytest.mark.parametrize("n", [1, 3])
def test_a_solve_that_never_ends_reports_its_last_residual(lib, n):
    """The host stops a solve whose device never reports an end; the residual it returns is that of the
    last FP64 update, not 0."""
    reset(lib)
    g = Host(lib, (4, 4, 4, 4))
    script(lib, 0.3, 0.0, 0.0, 0.0, 0.0)
    lib.fake_ignore_maxit()
    p = g.params(max_iter=10)
    code, st = g.batch(p, n) if n > 1 else g.solve(p)
    assert code == NOCONV
    assert all(s.status == NOCONV and s.reliable_updates > 0 and s.true_rel_res > 0 for s in st)
    reset(lib)
    g.close()
