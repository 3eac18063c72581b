"""FP64 operators on both parities in one launch: wd_apply and wd_apply_dag (on the caller's fields,
links that are not SU(3) too), and BiCGstab-M, whose final residuals take the full-lattice hop (forward
links only, the two parities' blocks in turn, blocks ordered t fastest in groups of a t-slice) on every
lattice and whose iteration does so above 16384 sites, here 8x16x36x4. Shapes at the edges of that order:
slices of 9 blocks (a smaller last group), of exactly one group, of one block, of no whole number of
blocks, T = 2, and the smallest lattice.

Tolerance: one application has about 150 rounded FP64 terms per component, of comparable size:
150 x 1.1e-16 < 2e-14 relative to the largest component.
"""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_1103_5103_amd as wd

pytestmark = pytest.mark.gpu
SHAPES = [(8, 16, 36, 4), (16, 16, 18, 2), (16, 16, 16, 2), (8, 8, 8, 4), (6, 10, 4, 6), (2, 2, 2, 2), (4, 4, 4, 8), (40, 2, 2, 4), (14, 10, 6, 2)]


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("su3", [True, False])
@pytest.mark.parametrize("dims", SHAPES)
def test_apply_matches_oracle(dims, su3):
    print("case", dims, su3, flush=True)
    anti = dims[0] != 6
    U = li.random_links(dims, 1.0, 1901)
    if not su3:
        U = U + 0.1 * li.random_links(dims, 0.3, 1902)
    psi = li.gaussian_field(dims, 2901)
    g = wd.wd_gauge_create(_t(U), antiperiodic=anti)
    for dag in (False, True):
        ref = oracle.apply(U, 0.125, psi, dag=dag, antiperiodic=anti)
        out = (wd.wd_apply_dag if dag else wd.wd_apply)(g, 0.125, _t(psi)).cpu().numpy()
        assert np.abs(out - ref).max() <= 2e-14 * np.abs(ref).max(), (dims, su3, dag)
    g.close()


@pytest.mark.parametrize("dims", SHAPES[:5])
@pytest.mark.parametrize("gauge", ["caller", "temporal"])
def test_bicgstab_m_matches_oracle(dims, gauge):
    print("case", dims, gauge, flush=True)
    kappas = [0.12, 0.13]
    U, b = li.random_links(dims, 1.0, 1903), li.gaussian_field(dims, 2903)
    p = wd.params(tol=1e-10, mixed=False, eo=False)
    g = wd.wd_gauge_create(_t(U), hint=wd.params(mixed=False, temporal_gauge=gauge == "temporal", nonchiral=gauge == "caller"))
    xs, sts = wd.bicgstab_m_solve(g, kappas, _t(b), p=p)
    for k, x, s in zip(kappas, xs, sts):
        res = oracle.true_residual(U, k, x.cpu().numpy(), b)
        assert res < 1e-10 and abs(res - s["true_rel_res"]) < 1e-3 * res + 1e-15, (dims, k, res, s)
    g.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (8, 16, 36, 4)])
def test_apply_with_overlapping_fields(dims):
    """Distinct in and out that share memory give the result of separate fields."""
    U = li.random_links(dims, 1.0, 1905)
    g = wd.wd_gauge_create(_t(U))
    n = int(np.prod(g.field_shape))
    for dag in (False, True):
        for shift in (1, n // 2):
            buf = torch.zeros(n + shift, dtype=torch.complex128, device="cuda")
            psi = _t(li.gaussian_field(dims, 2905))
            ref = (wd.wd_apply_dag if dag else wd.wd_apply)(g, 0.12, psi)
            for no_alloc in (False, True):
                a, b = buf[:n].view(g.field_shape), buf[shift:].view(g.field_shape)
                b.copy_(psi)
                if no_alloc:
                    wd.wd_apply_noalloc(g, 0.12, b, a, dagger=dag)
                else:
                    (wd.wd_apply_dag if dag else wd.wd_apply)(g, 0.12, b, out=a)
                assert torch.equal(a, ref), (dims, dag, shift, no_alloc)
    g.close()
