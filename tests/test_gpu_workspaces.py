"""A handle's workspaces are parts of a few allocations, made when a solver first needs them. One handle
that goes through every solver, in changing formats and with changing numbers of masses, gives bit for
bit what a handle of its own gives for each call, and holds no more than before when a call comes again.
"""
import pytest
import torch

import lattice_inputs as li
import paper_1103_5103_amd as wd

pytestmark = pytest.mark.gpu
KAPPAS = [0.120, 0.124, 0.127]


def _calls(b):
    f32, f16 = wd.params(tol=1e-8), wd.params(tol=1e-8, spinor="f16", links="f16")
    f64 = wd.params(tol=1e-8, mixed=False)
    out = []
    for p in (f32, f16, f64):
        out.append(lambda g, p=p: [wd.bicgstab_solve(g, 0.125, b, p=p)[0]])
        for n in (1, 3):
            out.append(lambda g, p=p, n=n: wd.wd_multimass_solve(g, KAPPAS[:n], b, p=p)[0])
        out.append(lambda g, p=p: wd.wd_normal_solve(g, 0.12, [0.0, 0.1], b, p=p)[0])
    for n in (2, 3):
        out.append(lambda g, n=n: wd.bicgstab_m_solve(g, KAPPAS[:n], b, p=f64)[0])
        out.append(lambda g, n=n: wd.wd_normal_solve(g, 0.12, [0.0, 0.1, 0.2][:n], b,
                                                     method=wd.WD_METHOD_MULTISHIFT, p=f64)[0])
    return out


@pytest.mark.parametrize("opts", [{}, {"temporal_gauge": True}, {"links": "bf16"}])
@pytest.mark.parametrize("dims", [(2, 4, 6, 4), (8, 8, 8, 8)])
def test_one_handle_for_every_solver(dims, opts):
    print("case", dims, opts, flush=True)
    U = torch.from_numpy(li.random_links(dims, 0.4, 77)).cuda()
    b = torch.from_numpy(li.gaussian_field(dims, 78)).cuda()
    hint = wd.params(**opts)
    calls = _calls(b)
    want = []
    for f in calls:
        g = wd.wd_gauge_create(U, hint=hint)
        want.append([x.clone() for x in f(g)])
        g.close()
    g = wd.wd_gauge_create(U, hint=hint)
    held = []
    for rounds in range(3):
        for f, w in zip(calls, want):
            for x, y in zip(f(g), w):
                assert torch.equal(x, y)
        held.append(g.device_bytes())
    assert held[1] == held[2]
    g.close()
