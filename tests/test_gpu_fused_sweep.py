"""Solves whose launches have more than 1024 blocks form delta and alpha of an iteration from the second
hop's sums, before the sweep that updates x, r and s. They must come as far as solves that sum delta
from the residual: links and masses with slow, uneven convergence, in FP64 to the last digits.

On the CPU (FP64, tree-ordered sums; delta summed from the residual / formed as here / formed from
<rhat, A w> alone): M_prec on 8^4, eps 0.3, kappa 0.13 reaches 1e-11 in 60 / 60 / more than 200 iterations.

Tolerances: the iterated residual is below tol when a solve ends; each iteration rounds x and r in about
30 operations, so the true residual is within 30 x 1.1e-16 x iterations of it (relative to |b|).
"""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_1103_5103_amd as wd

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _bound(tol, iters):
    return tol + 30 * 1.1e-16 * iters


@pytest.mark.parametrize("kappa,tol", [(0.134, 1e-13), (0.134, 1e-14), (0.2, 1e-13), (0.2, 1e-14)])
def test_bicgstab_m_reaches_small_residuals(kappa, tol):
    dims = (16, 16, 16, 72)  # 1152 blocks of both parities
    print("case", dims, kappa, tol, flush=True)
    U, b = li.random_links(dims, 1.0, 2001), li.gaussian_field(dims, 3001)
    g = wd.wd_gauge_create(_t(U))
    kappas = [kappa, 0.9 * kappa]
    xs, sts = wd.bicgstab_m_solve(g, kappas, _t(b), p=wd.params(tol=tol, mixed=False, eo=False, max_iter=120),
                                  raise_on_fail=False)
    print(sts, flush=True)
    for k, x, s in zip(kappas, xs, sts):
        assert s["status"] == 0
        assert oracle.true_residual(U, k, x.cpu().numpy(), b) < _bound(tol, s["iters"])
    g.close()


@pytest.mark.parametrize("dims,n,kappa,tol,max_iter", [((8, 8, 8, 8), 130, 0.13, 1e-11, 120), ((12, 12, 12, 12), 26, 0.134, 1e-10, 1000)])
def test_batch_reaches_small_residuals(dims, n, kappa, tol, max_iter):
    print("case", dims, n, kappa, tol, flush=True)
    U = li.random_links(dims, 0.3, 7)
    src = [li.gaussian_field(dims, 8 + k) for k in range(3)]
    g = wd.wd_gauge_create(_t(U))
    p = wd.params(tol=tol, mixed=False, max_iter=max_iter)
    b = [_t(v) for v in src]
    x = [torch.empty_like(b[0]) for _ in range(n)]
    sts = wd.wd_batch_solve([(g, kappa, b[i % 3], x[i]) for i in range(n)], p=p, raise_on_fail=False)
    one = [wd.bicgstab_solve(g, kappa, v, p=p, raise_on_fail=False)[1] for v in b]  # delta from the residual
    print([s["iters"] for s in one], sorted({(i % 3, s["iters"], s["status"]) for i, s in enumerate(sts)}), flush=True)
    assert all(s["status"] == 0 for s in sts + one)
    for i in range(3):
        assert oracle.true_residual(U, kappa, x[i].cpu().numpy(), src[i]) < _bound(tol, sts[i]["iters"])
    g.close()
