"""The hop for small launches (one system, at most 16384 sites of one parity) and the finishers that
small launches fold into the following sweep, at the sizes around their limits: one block, a block of
few sites, the largest lattice of the small hop and the next one; every storage format, both methods of
mixed precision, the adjoint solve, the temporal gauge; a whole solve against the oracle's residual and
the operator site by site (tolerances of the storage formats: unit roundoff times about a dozen terms).
"""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_1103_5103_amd as wd

pytestmark = pytest.mark.gpu
SHAPES = [(2, 2, 2, 2), (4, 4, 4, 8), (6, 2, 10, 4), (16, 16, 16, 8), (16, 16, 16, 10)]
FORMATS = [("f64", "f64"), ("f32", "f16"), ("f32", "bf16"), ("f32", "f32"), ("f16", "f16")]
SITE_TOL = {"f64": 1e-13, "f32f32": 1e-6, "f32f16": 1e-2, "f32bf16": 2e-2, "f16f16": 1e-2}


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _params(spinor, links, **kw):
    return wd.params(mixed=False, **kw) if spinor == "f64" else wd.params(spinor=spinor, links=links, **kw)


@pytest.mark.parametrize("spinor,links", FORMATS)
@pytest.mark.parametrize("dims", SHAPES)
def test_operator(dims, spinor, links):
    print("case", dims, spinor, links, flush=True)
    U, psi = li.random_links(dims, 1.0, 1951), li.gaussian_field(dims, 2951)
    even = oracle.even_part(psi)
    for opts in ({}, {"nonchiral": True}, {"temporal_gauge": True}):
        p = _params(spinor, links, **opts)
        g = wd.wd_gauge_create(_t(U), hint=p)
        for red in ("none", "zdot", "outx", "norm"):
            out, dots = wd.wd_apply_prec(g, 0.13, _t(psi), p=p, v=wd.op_variant(red=red))
            ref = oracle.mprec(U, 0.13, even)
            e = oracle.even_part(out.cpu().numpy())
            scale = np.sqrt((np.abs(ref) ** 2).sum() / (ref.size / 24))
            err = np.sqrt((np.abs(e - ref) ** 2).sum(axis=(-1, -2))).max() / scale
            assert err < SITE_TOL["f64" if spinor == "f64" else spinor + links], (dims, opts, red, err)
            if red == "zdot":
                want = np.vdot(even, ref)
                assert abs(complex(dots[0][0], dots[0][1]) - want) < 2e-2 * abs(want)
        g.close()


@pytest.mark.parametrize("spinor,links", FORMATS)
@pytest.mark.parametrize("dims", SHAPES)
def test_solve(dims, spinor, links):
    print("case", dims, spinor, links, flush=True)
    U, b = li.random_links(dims, 1.0, 1952), li.gaussian_field(dims, 2952)
    for kw in (dict(delta=0.1), dict(delta=1e-3, defect_correction=True), dict(delta=0.1, dagger=True)):
        p = _params(spinor, links, tol=1e-9, **kw)
        g = wd.wd_gauge_create(_t(U), hint=p)
        x, st = wd.bicgstab_solve(g, 0.125, _t(b), p=p)
        r = b - oracle.apply(U, 0.125, x.cpu().numpy(), dag=bool(kw.get("dagger")))
        assert st["status"] == 0 and np.linalg.norm(r) < 1e-9 * np.linalg.norm(b), (dims, kw, st)
        g.close()


@pytest.mark.parametrize("spinor,links", [("f64", "f64"), ("f32", "f16"), ("f16", "f16")])
def test_solve_above_the_folded_sizes(spinor, links):
    """Just above the launches with folded finishers (294912 sites per parity, 1152 blocks): the
    second hop's sums give alpha, and one sweep updates x, r and s."""
    dims = (32, 32, 32, 18)
    U, b = li.random_links(dims, 1.0, 1961), li.gaussian_field(dims, 2961)
    g = wd.wd_gauge_create(_t(U), hint=_params(spinor, links))
    for kw in (dict(delta=0.1), dict(delta=1e-3, defect_correction=True)):
        p = _params(spinor, links, tol=1e-9, **kw)
        x, st = wd.bicgstab_solve(g, 0.13, _t(b), p=p)
        res = oracle.true_residual(U, 0.13, x.cpu().numpy(), b)
        print(spinor, kw, st, res, flush=True)
        assert st["status"] == 0 and res < 1e-9
        if spinor == "f64":
            xs, sts = wd.bicgstab_m_solve(g, [0.13, 0.12], _t(b), p=wd.params(tol=1e-9, mixed=False, eo=False))
            assert all(oracle.true_residual(U, k, x.cpu().numpy(), b) < 1e-9 for k, x in zip([0.13, 0.12], xs))
            break
    g.close()
