"""The shifted systems of BiCGstab-M and CG-M are updated once per block of iterations. A solve that
is stopped after a given number of iterations (inside the first block, at its end, one past it, in
and at the end of the second, one past it) must hold the same iterates as the oracle, which updates them in every
iteration; some shifts freeze inside a block. Also without shifts, with a repeated mass and with a
zero source.

Tolerance: the two differ by the rounding of about 17 FP64 iterations whose coefficients amplify it
by less than 1e3: 17 x 1e3 x 2.2e-16 < 1e-11.
"""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_1103_5103_amd as wd

pytestmark = pytest.mark.gpu
DIMS = (8, 4, 6, 4)
KAPPAS = [0.134, 0.12, 0.08, 0.134, 0.05, 0.128, 0.03, 0.11, 0.1]
SIGMAS = [25.0, 0.0, 400.0, 100.0, 0.0, 1600.0, 6400.0, 800.0, 50.0]
STOPS = [1, 2, 7, 8, 9, 15, 16, 17]


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _close(x, ref):
    return np.linalg.norm(x.cpu().numpy() - ref) <= 1e-11 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [1, 2, 9])
def test_bicgstab_m_iterates(n):
    U, b = li.random_links(DIMS, 1.0, 1801), li.gaussian_field(DIMS, 2801)
    g = wd.wd_gauge_create(_t(U))
    for stop in STOPS:
        p = wd.params(tol=1e-6, mixed=False, eo=False, max_iter=stop)
        xs, sts = wd.bicgstab_m_solve(g, KAPPAS[:n], _t(b), p=p, raise_on_fail=False)
        ref, it, _, conv = oracle.bicgstab_m(U, KAPPAS[:n], b, tol=1e-6, maxit=stop)
        print("n", n, "stop", stop, [s["iters"] for s in sts], conv, flush=True)
        assert max(s["iters"] for s in sts) == it
        for x, r in zip(xs, ref):
            assert _close(x, r), (n, stop)
    g.close()


@pytest.mark.parametrize("n", [1, 3, 9])
def test_cg_m_iterates(n):
    U, b = li.random_links(DIMS, 1.0, 1802), li.gaussian_field(DIMS, 2802)
    g = wd.wd_gauge_create(_t(U), hint=wd.params(nonchiral=True))
    for stop in STOPS:
        p = wd.params(tol=1e-6, mixed=False, max_iter=stop)
        xs, sts = wd.wd_normal_solve(g, 0.134, SIGMAS[:n], _t(b), method=wd.WD_METHOD_MULTISHIFT, p=p, raise_on_fail=False)
        ref, it, _, conv = oracle.cg_m(U, 0.134, SIGMAS[:n], b, tol=1e-6, maxit=stop)
        print("n", n, "stop", stop, [s["iters"] for s in sts], conv, flush=True)
        assert max(s["iters"] for s in sts) == it
        for x, r in zip(xs, ref):
            assert _close(x, r), (n, stop)
    g.close()


def test_zero_source_after_a_solve():
    U, b = li.random_links(DIMS, 1.0, 1803), li.gaussian_field(DIMS, 2803)
    g = wd.wd_gauge_create(_t(U))
    z = torch.zeros(g.field_shape, dtype=torch.complex128, device="cuda")
    p = wd.params(tol=1e-8, mixed=False, eo=False)
    for field in (_t(b), z):
        xs, _ = wd.bicgstab_m_solve(g, KAPPAS, field, p=p)
        ys, _ = wd.wd_normal_solve(g, 0.134, SIGMAS, field, method=wd.WD_METHOD_MULTISHIFT, p=p)
    assert all(float(x.abs().max()) == 0.0 for x in xs + ys)
    g.close()


def test_graph_replays():
    U, b = li.random_links(DIMS, 1.0, 1804), li.gaussian_field(DIMS, 2804)
    g = wd.wd_gauge_create(_t(U))
    p = wd.params(tol=1e-10, mixed=False, eo=False)

    def solve(n):
        xs, _ = wd.bicgstab_m_solve(g, KAPPAS[:n], _t(b), p=p)
        ys, _ = wd.wd_normal_solve(g, 0.134, SIGMAS[:n], _t(b), method=wd.WD_METHOD_MULTISHIFT, p=p)
        return xs + ys

    ref = {n: solve(n) for n in (3, 9)}
    wd.set_graphs(True)
    try:
        for n in (3, 9, 3, 9, 3):  # more shifts need larger buffers than those first captured
            assert all(torch.equal(x, r) for x, r in zip(solve(n), ref[n])), n
    finally:
        wd.set_graphs(False)
        g.close()
