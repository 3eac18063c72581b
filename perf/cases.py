"""The work that a user of wdirac has it do: operator applications, solves for one and several
masses, batches of systems, the normal equations, and differentiation, each through the public entry
points. listed() names fixed cases, draw() gives more of the same ranges, prepare() makes what a
program holds before the call, run() is one call, work() the bytes and operations it cannot do
without, exact() the result in 64 bits from plain torch.

Inputs are near-Haar random SU(3) links exp(i eps H) and Gaussian or point sources, as in
lattice_inputs and the benchmark. Solves run to 1e-10, the accuracy of the paper's Table 3 (1e-11
where gradients are formed from them).
"""
import math

import torch

DEV = "cuda"

TOL = 1e-10
TOL_GRAD = 1e-11


def listed():
    return [
        # One operator application on the smallest lattice of the tests: a Krylov method of the
        # user's own, or a check of a residual, where latency and launches are all there is.
        dict(name="apply_4x8", kind="apply", X=4, Y=4, Z=4, T=8, eps=0.3, anti=True, dagger=False),
        # The adjoint operator on a mid-size production lattice.
        dict(name="apply_dag_24x48", kind="apply", X=24, Y=24, Z=24, T=48, eps=1.0, anti=True, dagger=True),
        # One mass on a small lattice with the default storage (FP32 spinors, FP16 12-real links).
        dict(name="solve_8", kind="solve", X=8, Y=8, Z=8, T=8, eps=1.0, anti=True, kappa=0.125, spinor="f32",
             links="f16", recon=12, delta=0.1, defect=False, nonchiral=False, tgauge=False, dagger=False, source="gauss"),
        # One mass in FP64 throughout on a lattice of uneven extents, adjoint, periodic in time.
        dict(name="solve_f64_ragged", kind="solve", X=10, Y=6, Z=14, T=18, eps=1.0, anti=False, kappa=0.12,
             spinor="f64", links="f64", recon=12, delta=0.1, defect=False, nonchiral=False, tgauge=False, dagger=True,
             source="point"),
        # The small multi-mass workload of the benchmark: 16^3x32, six masses one after the other
        # with the extrapolated start guess, 16-bit storage.
        dict(name="masses_seq_16x32", kind="masses", method="sequential", X=16, Y=16, Z=16, T=32, eps=1.0, anti=True,
             kappa0=0.120, dkappa=0.002, n=6, spinor="f16", links="f16", delta=3e-3, defect=False, nonchiral=True),
        # The benchmark's headline solve: 32^3x64, eight masses in sequence.
        dict(name="masses_seq_32x64", kind="masses", method="sequential", X=32, Y=32, Z=32, T=64, eps=1.0, anti=True,
             kappa0=0.120, dkappa=0.002, n=8, spinor="f32", links="f16", delta=1e-3, defect=False, nonchiral=True),
        # All masses of a source iterating together, BF16 links, the paper's defect correction.
        dict(name="masses_batched_24x48", kind="masses", method="batched", X=24, Y=24, Z=24, T=48, eps=1.0, anti=True,
             kappa0=0.120, dkappa=0.002, n=6, spinor="f32", links="bf16", delta=1e-3, defect=True, nonchiral=False),
        # BiCGstab-M (FP64) on both of the benchmark's lattices: the method the paper compares with.
        dict(name="masses_shift_16x32", kind="masses", method="multishift", X=16, Y=16, Z=16, T=32, eps=1.0, anti=True,
             kappa0=0.120, dkappa=0.002, n=6, spinor="f64", links="f64", delta=0.1, defect=False, nonchiral=False),
        dict(name="masses_shift_32x64", kind="masses", method="multishift", X=32, Y=32, Z=32, T=64, eps=1.0, anti=True,
             kappa0=0.120, dkappa=0.002, n=8, spinor="f64", links="f64", delta=0.1, defect=False, nonchiral=True),
        # A propagator's sources and masses at once on lattices of several sizes: 12 spin-colour
        # point sources x 4 masses on 16^3x32 and 4 x 4 on each of 8^4, 12^4, 16^4.
        dict(name="batch_sources", kind="batch", X=16, Y=16, Z=16, T=32, eps=1.0, anti=True, sources=12, kappa0=0.124,
             dkappa=0.002, n=4, uneven=True, spinor="f16", links="f16", delta=0.1, nonchiral=False),
        # A differentiable solve: new links in every step, so the handle is built in it, forward
        # and backward, gradients of the links and of the source.
        dict(name="train_16x32", kind="train", X=16, Y=16, Z=16, T=32, eps=1.0, anti=True, kappa=0.125, spinor="f32",
             links="f16", delta=0.1, force=False),
        # The shifted normal equations with CG-M, eight shifts as in the benchmark.
        dict(name="normal_shift_24x48", kind="normal", method="multishift", X=24, Y=24, Z=24, T=48, eps=1.0, anti=True,
             kappa=0.134, sigma_max=1600.0, n=8, spinor="f64", links="f64", delta=1e-3, nonchiral=False),
    ]


def _even(v, lo=4):
    return max(lo, 2 * int(round(v / 2)))


def draw(rng):
    """One more case: any kind, a volume between 4^3x8 and 32^3x64 (log-uniform), uneven extents."""
    cap = max(work(c)["bytes"] for c in listed())
    while True:
        v = math.exp(rng.uniform(math.log(512), math.log(32 ** 3 * 64)))
        side = v ** 0.25 * 0.85
        X, Y, Z = (min(48, _even(side * rng.uniform(0.7, 1.4))) for _ in range(3))
        T = min(96, _even(v / (X * Y * Z)))
        c = dict(kind=rng.choice(["apply", "solve", "masses", "masses", "batch", "train", "normal"]), X=X, Y=Y, Z=Z, T=T,
                 eps=1.0, anti=rng.random() < 0.8)
        spinor = rng.choice(["f32", "f32", "f16", "f64"])
        links = "f64" if spinor == "f64" else rng.choice(["f16", "f16", "bf16", "f32"])
        delta = rng.choice([0.1, 3e-3, 1e-3])
        nonchiral, defect = rng.random() < 0.5, rng.random() < 0.3
        if c["kind"] == "apply":
            c.update(dagger=rng.random() < 0.5, eps=rng.choice([0.3, 1.0]))
        elif c["kind"] == "solve":
            c.update(kappa=round(rng.uniform(0.115, 0.134), 4), spinor=spinor, links=links, recon=12, delta=delta,
                     defect=defect, nonchiral=nonchiral, tgauge=rng.random() < 0.2, dagger=rng.random() < 0.4,
                     source=rng.choice(["gauss", "point"]))
            if c["links"] == "f16" and not c["tgauge"] and rng.random() < 0.2:
                c["recon"] = 8
        elif c["kind"] == "masses":
            n = rng.randint(2, 8)
            method = rng.choice(["sequential", "batched", "multishift", "multishift"])
            if method == "multishift":
                spinor = links = "f64"
            c.update(method=method, n=n, kappa0=round(rng.uniform(0.115, 0.120), 4), dkappa=0.002, spinor=spinor, links=links,
                     delta=delta, defect=defect, nonchiral=nonchiral)
        elif c["kind"] == "batch":
            c.update(sources=rng.randint(2, 12), n=rng.randint(1, 4), kappa0=0.124, dkappa=0.002, uneven=rng.random() < 0.4,
                     spinor=spinor, links=links, delta=delta, nonchiral=nonchiral)
        elif c["kind"] == "train":
            c.update(kappa=round(rng.uniform(0.115, 0.13), 4), spinor=spinor, links=links, delta=delta,
                     force=rng.random() < 0.5)
        else:
            method = rng.choice(["multishift", "sequential"])
            if method == "multishift":
                spinor = links = "f64"
            c.update(method=method, n=rng.randint(2, 8), kappa=round(rng.uniform(0.12, 0.134), 4),
                     sigma_max=rng.choice([400.0, 1600.0]), spinor=spinor, links=links, delta=delta, nonchiral=nonchiral)
        if work(c)["bytes"] <= cap and c["X"] * c["Y"] * c["Z"] * c["T"] <= 32 ** 3 * 64:
            return c


# ---------------------------------------------------------------- inputs

def _dims(c):
    return c["X"], c["Y"], c["Z"], c["T"]


def _lattices(c):
    """(dims, number of sources) of a batch."""
    out = [(_dims(c), c["sources"])]
    if c["uneven"]:
        out += [((k, k, k, k), 4) for k in (8, 12, 16)]
    return out


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _gauss(gen, shape):
    return torch.randn(*shape, dtype=torch.complex128, device=DEV, generator=gen)


def _links(dims, eps, gen, chunk=1 << 20):
    """exp(i eps H), H traceless Hermitian Gaussian, shape [4, T, Z, Y, X, 3, 3]."""
    X, Y, Z, T = dims
    n = 4 * X * Y * Z * T
    out = torch.empty(n, 3, 3, dtype=torch.complex128, device=DEV)
    eye = torch.eye(3, dtype=torch.complex128, device=DEV)
    for lo in range(0, n, chunk):
        m = min(chunk, n - lo)
        g = _gauss(gen, (m, 3, 3))
        h = 0.5 * (g + g.mH.contiguous())
        h = h - (torch.diagonal(h, dim1=-2, dim2=-1).sum(-1) / 3.0)[:, None, None] * eye
        a = h * (1j * eps / 32.0)
        e = eye + a / 12.0
        for k in range(11, 0, -1):  # Taylor series of the exponential (Horner), then squarings
            e = eye + torch.bmm(a, e) / k
        for _ in range(5):
            e = torch.bmm(e, e)
        out[lo:lo + m] = e
    return out.reshape(4, T, Z, Y, X, 3, 3)


def _field(dims, gen):
    X, Y, Z, T = dims
    return _gauss(gen, (T, Z, Y, X, 3, 4))


def _point(dims, spin, colour, place):
    X, Y, Z, T = dims
    b = torch.zeros(T, Z, Y, X, 3, 4, dtype=torch.complex128, device=DEV)
    p = place % (X * Y * Z * T)
    b.view(-1, 3, 4)[p, colour, spin] = 1.0
    return b


def _inputs(c, seed):
    """The links and fields of a case, from the seed alone: a list of (dims, U, [fields])."""
    gen = _gen(seed)
    if c["kind"] == "batch":
        out = []
        for dims, ns in _lattices(c):
            U = _links(dims, c["eps"], gen)
            out.append((dims, U, [_point(dims, s % 4, (s // 4) % 3, seed * 977 + 31 * s) for s in range(ns)]))
        return out
    dims = _dims(c)
    U = _links(dims, c["eps"], gen)
    if c["kind"] == "solve" and c["source"] == "point":
        return [(dims, U, [_point(dims, seed % 4, seed % 3, seed * 977)])]
    return [(dims, U, [_field(dims, gen) for _ in range(2 if c["kind"] == "train" else 1)])]


def _kappas(c):
    return [round(c["kappa0"] + c["dkappa"] * i, 6) for i in range(c["n"])]


def _sigmas(c):
    """0 and a geometric series up to sigma_max: 0, 25, 50, ... for 1600 and 8 shifts."""
    n = c["n"]
    return [0.0] + [c["sigma_max"] / 2.0 ** (n - 2 - i) for i in range(n - 1)]


def _params(c, tol=TOL):
    import paper_1103_5103_amd as wd

    if c["spinor"] == "f64":
        return wd.params(tol=tol, mixed=False, nonchiral=c.get("nonchiral", False), temporal_gauge=c.get("tgauge", False),
                         dagger=c.get("dagger", False))
    return wd.params(tol=tol, spinor=c["spinor"], links=c["links"], recon=c.get("recon", 12), delta=c["delta"],
                     defect_correction=c.get("defect", False), nonchiral=c.get("nonchiral", False),
                     temporal_gauge=c.get("tgauge", False), dagger=c.get("dagger", False))


def prepare(case, seed):
    import paper_1103_5103_amd as wd

    kind = case["kind"]
    data = _inputs(case, seed)
    dims, U, fields = data[0]
    if kind == "apply":
        g = wd.wd_gauge_create(U, antiperiodic=case["anti"])
        return dict(case=case, g=g, psi=fields[0], out=torch.empty_like(fields[0]))
    if kind == "train":
        return dict(case=case, U=U.requires_grad_(True), b=fields[0].requires_grad_(True), eta=fields[1],
                    p=_params(case, TOL_GRAD))
    p = _params(case)
    if kind == "batch":
        systems, xs, gs = [], [], []
        ks = _kappas(case)
        for dims, U, bs in data:
            g = wd.wd_gauge_create(U, antiperiodic=case["anti"], hint=p)
            x = torch.zeros(len(bs) * len(ks), *g.field_shape, dtype=torch.complex128, device=DEV)
            gs.append(g)
            xs.append(x)
            for i, b in enumerate(bs):
                for j, k in enumerate(ks):
                    systems.append((g, k, b, x[i * len(ks) + j]))
        return dict(case=case, systems=systems, xs=xs, gs=gs, p=p)
    g = wd.wd_gauge_create(U, antiperiodic=case["anti"], hint=p)
    if kind == "masses" and case["method"] == "multishift":
        p = wd.params(tol=TOL, mixed=False, eo=False)
    return dict(case=case, g=g, b=fields[0], p=p)


def run(state):
    import paper_1103_5103_amd as wd

    c = state["case"]
    kind = c["kind"]
    if kind == "apply":
        f = wd.wd_apply_dag if c["dagger"] else wd.wd_apply
        return f(state["g"], 0.125, state["psi"], out=state["out"])
    if kind == "solve":
        return wd.bicgstab_solve(state["g"], c["kappa"], state["b"], p=state["p"])[0]
    if kind == "masses":
        if c["method"] == "multishift":
            return wd.bicgstab_m_solve(state["g"], _kappas(c), state["b"], p=state["p"])[0]
        m = wd.WD_METHOD_SEQUENTIAL if c["method"] == "sequential" else wd.WD_METHOD_BATCHED
        return wd.wd_multimass_solve(state["g"], _kappas(c), state["b"], method=m, p=state["p"])[0]
    if kind == "batch":
        wd.wd_batch_solve(state["systems"], p=state["p"])
        return state["xs"]
    if kind == "normal":
        m = wd.WD_METHOD_SEQUENTIAL if c["method"] == "sequential" else wd.WD_METHOD_MULTISHIFT
        return wd.wd_normal_solve(state["g"], c["kappa"], _sigmas(c), state["b"], method=m, p=state["p"])[0]
    x = wd.wilson_solve(state["U"], state["b"], c["kappa"], params=state["p"], antiperiodic=c["anti"],
                        project_su3=c["force"])
    gU, gb = torch.autograd.grad(x, (state["U"], state["b"]), grad_outputs=state["eta"])
    return dict(x=x.detach(), grad_U=gU, grad_b=gb)


# ---------------------------------------------------------------- what a pass cannot do without

FLOPS_HOP = 1320.0  # floating-point operations of the hopping term per site (both parities)


def work(case):
    """Bytes and operations per pass. An operator application in storage of s bytes a real and l
    bytes a link real reads the spinor and the 4 links of every site once and writes the spinor. A
    solve makes its iterations (estimated from kappa and the tolerance; every BiCGstab iteration
    takes two operator applications and reads and writes x, r and s once), reads its source and
    links and writes its solutions."""
    c = case
    s, l = {"f64": (8, 8), "f32": (4, 2), "f16": (2, 2)}[c.get("spinor", "f64")]
    if c.get("links") == "f32":
        l = 4
    V = c["X"] * c["Y"] * c["Z"] * c["T"]
    field64 = V * 24 * 8.0
    if c["kind"] == "apply":
        return {"bytes": 2 * field64 + V * 4 * 18 * 8.0, "flops": V * (FLOPS_HOP + 48)}
    digits = -math.log10(TOL_GRAD if c["kind"] == "train" else TOL)

    def iters(kappa, eo):
        # the hopping part shrinks a residual by about (2 kappa)^2 x 4 per application pair
        return math.ceil(digits * (1.0 if eo else 2.0) * kappa / 0.134)

    # an application of the even-odd operator: both hops, each link of the lattice read once by each
    eo_app = V * (2 * 24 * s + 4 * 12 * l)
    if c["kind"] == "solve":
        it = iters(c["kappa"], True)
        return {"bytes": it * (2 * eo_app + 3 * V * 24 * s) + 2 * field64, "flops": it * 2 * V * FLOPS_HOP}
    if c["kind"] == "masses":
        if c["method"] == "multishift":
            it = iters(c["kappa0"] + c["dkappa"] * (c["n"] - 1), False)
            per = 2 * (2 * field64 + V * 4 * 12 * 8.0) + 6 * field64
            return {"bytes": it * per + (1 + c["n"]) * field64, "flops": it * 2 * V * FLOPS_HOP}
        it = sum(iters(k, True) for k in _kappas(c)) * (0.6 if c["method"] == "sequential" else 1.0)
        return {"bytes": it * (2 * eo_app + 3 * V * 24 * s) + (1 + c["n"]) * field64, "flops": it * 2 * V * FLOPS_HOP}
    if c["kind"] == "batch":
        by = fl = 0.0
        for (X, Y, Z, T), ns in _lattices(c):
            v = X * Y * Z * T
            it = sum(iters(k, True) for k in _kappas(c)) * ns
            by += it * (2 * v * (2 * 24 * s) + 3 * v * 24 * s) + ns * (1 + c["n"]) * v * 192.0
            fl += it * 2 * v * FLOPS_HOP
        return {"bytes": by, "flops": fl}
    if c["kind"] == "train":
        it = 2 * iters(c["kappa"], True)
        return {"bytes": it * (2 * eo_app + 3 * V * 24 * s) + 4 * field64 + 2 * V * 4 * 18 * 8.0,
                "flops": it * 2 * V * FLOPS_HOP}
    it = math.ceil(digits * 2.5) * (1.0 if c["method"] == "multishift" else 0.6 * c["n"])
    return {"bytes": it * (2 * eo_app + 1.5 * V * 24 * s) + (0.5 + c["n"]) * field64, "flops": it * 2 * V * FLOPS_HOP}


# ---------------------------------------------------------------- the same in plain torch, 64 bits

def _gammas():
    """The chiral gamma matrices that multiply the 3x4 site matrix from the right."""
    g = torch.zeros(4, 4, 4, dtype=torch.complex128)
    g[0, 0, 3], g[0, 1, 2], g[0, 2, 1], g[0, 3, 0] = 1j, 1j, -1j, -1j
    g[1, 0, 3], g[1, 1, 2], g[1, 2, 1], g[1, 3, 0] = 1, -1, -1, 1
    g[2, 0, 2], g[2, 1, 3], g[2, 2, 0], g[2, 3, 1] = 1j, -1j, -1j, 1j
    for a in range(4):
        g[3, a, (a + 2) % 4] = -1
    return g.to(DEV)


class _Dirac:
    """M(kappa), its hopping term and their adjoints on fields [T, Z, Y, X, 3, 4]."""

    def __init__(self, U, anti):
        self.U, self.Ud, self.anti = U, U.mH.contiguous(), anti
        eye, g = torch.eye(4, dtype=torch.complex128, device=U.device), _gammas()
        self.minus, self.plus = [eye - m for m in g], [eye + m for m in g]
        self.g5 = torch.tensor([1.0, 1.0, -1.0, -1.0], dtype=torch.float64, device=U.device)

    def shift(self, f, mu, step):
        """f(n + mu) for step = 1, f(n - mu) for step = -1, with the boundary sign in time."""
        d = 3 - mu
        r = torch.roll(f, -step, d)
        if mu == 3 and self.anti:
            r[-1 if step == 1 else 0] *= -1
        return r

    def hop(self, psi):
        out = torch.zeros_like(psi)
        shape = psi.shape
        for mu in range(4):
            f = torch.matmul(self.shift(psi, mu, 1).reshape(-1, 4), self.minus[mu]).reshape(-1, 3, 4)
            out += torch.bmm(self.U[mu].reshape(-1, 3, 3), f).reshape(shape)
            b = torch.bmm(self.Ud[mu].reshape(-1, 3, 3), torch.matmul(psi.reshape(-1, 4), self.plus[mu]).reshape(-1, 3, 4))
            out += self.shift(b.reshape(shape), mu, -1)
        return out

    def m(self, kappa, psi):
        return psi / (2.0 * kappa) - 0.5 * self.hop(psi)

    def m_dag(self, kappa, psi):
        return self.g5 * self.m(kappa, self.g5 * psi)


def _dot(a, b):
    return torch.sum(torch.conj(a) * b)


def _bicgstab(op, b, tol=2e-13, most=400):
    # a random shadow vector: with the residual itself a point source breaks down at once
    x, r = torch.zeros_like(b), b.clone()
    rh, p = _gauss(_gen(1), b.shape), r.clone()
    rho, bb = _dot(rh, r), float(_dot(b, b).real)
    for _ in range(most):
        v = op(p)
        a = rho / _dot(rh, v)
        s = r - a * v
        t = op(s)
        w = _dot(t, s) / _dot(t, t)
        x += a * p + w * s
        r = s - w * t
        if float(_dot(r, r).real) < tol * tol * bb:
            break
        rho2 = _dot(rh, r)
        p = r + (rho2 / rho) * (a / w) * (p - w * v)
        rho = rho2
    return x


def _cg(op, b, tol=2e-13, most=400):
    x, r = torch.zeros_like(b), b.clone()
    p, rr = r.clone(), float(_dot(b, b).real)
    bb = rr
    for _ in range(most):
        v = op(p)
        a = rr / float(_dot(p, v).real)
        x += a * p
        r -= a * v
        new = float(_dot(r, r).real)
        if new < tol * tol * bb:
            break
        p = r + (new / rr) * p
        rr = new
    return x


def _link_gradient(D, x, lam, force):
    shape = (-1, 3, 4)
    out = torch.empty_like(D.U)
    for mu in range(4):
        xs, ls = D.shift(x, mu, 1), D.shift(lam, mu, 1)
        g = torch.bmm(torch.matmul(lam.reshape(-1, 4), D.minus[mu]).reshape(shape), xs.reshape(shape).mH.contiguous())
        g += torch.bmm(torch.matmul(x.reshape(-1, 4), D.plus[mu]).reshape(shape), ls.reshape(shape).mH.contiguous())
        g *= 0.5
        if force:
            y = torch.bmm(D.U[mu].reshape(-1, 3, 3), g.mH.contiguous())
            a = 0.5 * (y - y.mH)
            tr = torch.diagonal(a, dim1=-2, dim2=-1).sum(-1) / 3.0
            g = 0.5j * (a - tr[:, None, None] * torch.eye(3, dtype=a.dtype, device=a.device))
        out[mu] = g.reshape(out[mu].shape)
    return out


def exact(case, seed):
    """The result of run() on the same inputs in 64 bits, by plain torch."""
    c = case
    data = _inputs(c, seed)
    dims, U, fields = data[0]
    if c["kind"] == "batch":
        out = []
        for dims, U, bs in data:
            D = _Dirac(U, c["anti"])
            out.append(torch.stack([_bicgstab(lambda v: D.m(k, v), b) for b in bs for k in _kappas(c)]))
        return out
    D = _Dirac(U, c["anti"])
    if c["kind"] == "apply":
        return (D.m_dag if c["dagger"] else D.m)(0.125, fields[0])
    if c["kind"] == "solve":
        op = D.m_dag if c["dagger"] else D.m
        return _bicgstab(lambda v: op(c["kappa"], v), fields[0])
    if c["kind"] == "masses":
        return [_bicgstab(lambda v: D.m(k, v), fields[0]) for k in _kappas(c)]
    if c["kind"] == "train":
        x = _bicgstab(lambda v: D.m(c["kappa"], v), fields[0])
        lam = _bicgstab(lambda v: D.m_dag(c["kappa"], v), fields[1])
        return dict(x=x, grad_U=_link_gradient(D, x, lam, c["force"]), grad_b=lam)
    X, Y, Z, T = dims
    t, z, y, x = torch.meshgrid(*(torch.arange(n, device=DEV) for n in (T, Z, Y, X)), indexing="ij")
    even = (((t + z + y + x) & 1) == 0)[..., None, None].to(torch.float64)
    a2 = (1.0 / (2.0 * c["kappa"])) ** 2

    def prec(v):
        return a2 * v - 0.25 * D.hop(D.hop(v))

    def normal(v):
        return D.g5 * prec(D.g5 * prec(v))

    b = even * fields[0]
    return [_cg(lambda v: normal(v) + s * v, b) for s in _sigmas(c)]
