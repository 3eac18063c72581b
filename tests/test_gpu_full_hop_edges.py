"""The full-lattice FP64 hop (both parities in one launch, forward links only) as BiCGstab-M's iteration
launches it: lattices of more than 16384 sites, below which the hop for small launches takes its place.
Its block order goes t fastest in groups of 8 blocks of a t-slice, or by sites where a slice is no whole
number of 256-site blocks; here: a smaller last group, exactly one group, one block a slice, T = 2, slices
of no whole number of blocks with a partial last block, each with the finishers folded into the sweeps (up
to 1024 blocks: the sums <z, out> and <out, x0>, |out|^2) and above (the second hop with all its sums).

Tolerances: the iterated residual is below 1e-10 at the end, rounding (30 operations x 1.1e-16 x 100 iterations)
stays below 4e-13. Two such solutions differ by at most 2 |M^-1| (1e-10 + 4e-13) |b|, and with links of norm 1 at
most |M x| >= (1/(2 kappa) - 4) |x|. The oracle's BiCGstab-M takes the same iterations, but for rounding at the
threshold.
"""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_1103_5103_amd as wd

pytestmark = pytest.mark.gpu
SHAPES = [
    (8, 16, 36, 8),     # 9 blocks a slice: a group of 8 and one of 1; 144 blocks
    (16, 16, 16, 6),    # one group of 8
    (8, 8, 8, 64),      # one block a slice
    (32, 16, 36, 2),    # T = 2
    (20, 14, 18, 6),    # 9.8 blocks a slice: site order, a partial last block; folded
    (20, 14, 18, 54),   # the same above 1024 blocks
    (16, 32, 36, 16),   # groups, above 1024 blocks
    (64, 64, 36, 2),    # T = 2, above 1024 blocks
]


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dims", SHAPES)
@pytest.mark.parametrize("opts", [dict(nonchiral=True), dict(temporal_gauge=True), dict(su3=False)])
def test_bicgstab_m_matches_oracle(dims, opts):
    print("case", dims, opts, flush=True)
    kappas = [0.118, 0.122]
    opts = dict(opts)
    U, b = li.random_links(dims, 1.0, 2011), li.gaussian_field(dims, 3011)
    if not opts.pop("su3", True):
        U = U * (1.0 - 2e-3 * np.random.default_rng(5).random(U.shape[:-2] + (1, 1)))  # 18-real links
    g = wd.wd_gauge_create(_t(U), hint=wd.params(mixed=False, **opts))
    xs, sts = wd.bicgstab_m_solve(g, kappas, _t(b), p=wd.params(tol=1e-10, mixed=False, eo=False))
    for k, x, s in zip(kappas, xs, sts):
        res = oracle.true_residual(U, k, x.cpu().numpy(), b)
        assert s["status"] == 0 and res < 1e-10 + 4e-13, (dims, k, res, s)
    if opts.get("nonchiral"):
        ref, iters, status, conv = oracle.bicgstab_m(U, kappas, b, tol=1e-10)
        assert status == 0 and abs(max(s["iters"] for s in sts) - iters) <= 1, (sts, iters)
        for k, x, r, s, c in zip(kappas, xs, ref, sts, conv):
            assert abs(s["iters"] - c) <= 1
            assert np.linalg.norm(x.cpu().numpy() - r) < 2 * (1e-10 + 4e-13) / (0.5 / k - 4) * np.linalg.norm(b)
    g.close()
