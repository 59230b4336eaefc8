"""Timed cases of the excess-chemical-potential evaluator: what a PNP-cDFT program has it do, through the
binding's public entry points, over the range of grid sizes, species counts, precisions and options it supports.

Inputs are synthetic electrolytes made on the GPU from a seed: charged hard spheres of 0.15-0.45 nm around a Gaussian
channel, with noise along every axis, so that every wave-vector carries data.

The mixed path computes in float32 and hands its results over in float64 storage; the programs that choose it keep them
as float32 fields (the accuracy they have), so the cases on that path end with that conversion, which is timed with them.
Every case also has its values in 64 bits (`exact`), from plain torch FFTs.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1407_0674_amd as pnp

FP64, MIXED = pnp.FP64, pnp.MIXED
ALL, HS, EC, SW, WB = pnp.TERM_ALL, pnp.TERM_HS, pnp.TERM_EC, pnp.TERM_SW, pnp.TERM_HS_WB
SIZES = (8, 16, 24, 32, 48, 64, 96, 128, 192, 256)
MOLAR = 0.602214076  # 1 mol/L in nm^-3


def listed():
    return [
        # one evaluation of a small cell (a parameter scan, a unit test of a solver): latency and launches
        dict(name="mu_fp64_16", kind="mu_ex", n=16, S=2, precision=FP64, terms=HS | SW, per_term=False, aperiodic=False),
        dict(name="mu_mixed_32", kind="mu_ex", n=32, S=3, precision=MIXED, terms=ALL, per_term=False, aperiodic=False),
        # a Gummel iteration's evaluation of a channel at ordinary sizes, in plain and in mixed precision
        dict(name="mu_fp64_64", kind="mu_ex", n=64, S=3, precision=FP64, terms=ALL, per_term=False, aperiodic=False),
        dict(name="mu_mixed_96_terms", kind="mu_ex", n=96, S=4, precision=MIXED, terms=ALL, per_term=True, aperiodic=False),
        dict(name="mu_fp64_128_wb", kind="mu_ex", n=128, S=3, precision=FP64, terms=WB | EC | SW, per_term=False, aperiodic=False),
        dict(name="mu_mixed_192", kind="mu_ex", n=192, S=2, precision=MIXED, terms=ALL, per_term=False, aperiodic=False),
        # the benchmark grid: the largest evaluation
        dict(name="mu_mixed_256", kind="mu_ex", n=256, S=3, precision=MIXED, terms=ALL, per_term=False, aperiodic=False),
        # a pore with walls: the non-periodic domain, through the doubled grid
        dict(name="mu_mixed_64_aperiodic", kind="mu_ex", n=64, S=3, precision=MIXED, terms=ALL, per_term=False, aperiodic=True),
        # a sweep of independent uneven cells in one batched call
        dict(name="batch_mixed", kind="batch", sizes="32,32,48,48,64,64,96,96,128,128", S=3, precision=MIXED),
        # resident states evaluated over and over: one captured replay per step
        dict(name="plan_mixed", kind="plan", sizes="48,64,64,96", S=3, precision=MIXED),
        # the initial state of a run: steps of the equilibrium solve
        dict(name="equilibrium_fp64_48", kind="equilibrium", n=48, S=2, precision=FP64, steps=10),
        # sphere integrals of a solver that works in real space
        dict(name="quad_mixed_192", kind="quad", nx=192, ny=192, nz=192, F=3, precision=MIXED, order=8, cubic=False, aperiodic=False),
    ]


def draw(rng):
    kind = rng.choice(["mu_ex"] * 6 + ["batch", "plan", "equilibrium", "quad", "quad", "weighted", "energy"])
    precision = rng.choice([FP64, MIXED])
    if kind == "mu_ex":
        aperiodic = rng.random() < 0.2
        per_term = rng.random() < 0.2
        top = (128 if precision == FP64 else 192) if not per_term else (96 if precision == FP64 else 128)
        n = rng.choice([v for v in SIZES if v <= top] + ([256] if precision == MIXED and not per_term else []))
        S = rng.randint(1, 3 if n >= 192 else 5 if n >= 96 else 8)
        terms = rng.choice([ALL, ALL, ALL, HS, HS | SW, EC | SW, WB | EC | SW])
        if aperiodic:
            n = rng.choice([v for v in (8, 12, 16, 24, 32, 48, 64) if 2 * v <= top])
        return dict(kind=kind, n=n, S=S, precision=precision, terms=terms, per_term=per_term, aperiodic=aperiodic)
    if kind in ("batch", "plan"):
        pool = (32, 48, 64, 96, 128) if precision == MIXED else (16, 24, 32, 48, 64)
        sizes = [rng.choice(pool) for _ in range(rng.randint(2, 8))]
        return dict(kind=kind, sizes=",".join(map(str, sizes)), S=rng.randint(2, 4), precision=precision)
    if kind == "equilibrium":
        return dict(kind=kind, n=rng.choice([16, 24, 32, 48, 64]), S=rng.randint(1, 3), precision=FP64, steps=rng.randint(3, 12))
    if kind == "quad":
        e = [max(7, round(math.exp(rng.uniform(math.log(16), math.log(160))))) for _ in range(3)]
        return dict(kind=kind, nx=e[0], ny=e[1], nz=e[2], F=rng.randint(1, 4), precision=precision,
                    order=rng.choice([4, 6, 8, 12]), cubic=rng.random() < 0.25, aperiodic=rng.random() < 0.3)
    n = rng.choice([16, 24, 32, 48, 64, 96])
    return dict(kind=kind, n=n, S=rng.randint(1, 4), precision=precision, terms=ALL)


# ---------------------------------------------------------------------------------------------------------------------
# inputs

def electrolyte(n, S, precision, terms, seed, h=0.05, packing=0.35):
    """(problem, rho): S species on an n^3 grid, all drawn from the seed."""
    r = np.random.default_rng(seed)
    d, q = r.uniform(0.15, 0.45, S), r.choice([-2.0, -1.0, 1.0, 2.0], S)
    rb = r.uniform(0.1, 1.0 if S > 4 else 2.0, S) * MOLAR
    L = n * h
    c, w = r.uniform(0.0, L, 2), r.uniform(L / 10, L / 6)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    x = torch.arange(n, device="cuda", dtype=torch.float64) * h
    dx, dz = ((x - v + 0.5 * L) % L - 0.5 * L for v in c)
    g = torch.exp(-(dx[:, None, None] ** 2 + dz[None, None, :] ** 2) / (2 * w * w))
    alt = 1.0 - 2.0 * (torch.arange(n, device="cuda", dtype=torch.float64) % 2)
    stag = (alt[:, None, None] + alt[None, :, None] + alt[None, None, :]) / 3
    rho = torch.rand((S, n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    eta = torch.zeros((), device="cuda", dtype=torch.float64)
    for i in range(S):
        rho[i] = rb[i] * (1 + 0.5 * np.sign(q[i]) * (2 * g - 1)) * (1 + 0.1 * (2 * rho[i] - 1) + 0.05 * stag)
        eta = eta + rho[i] * (math.pi / 6 * d[i] ** 3)
    f = min(1.0, packing / float(eta.max()))  # dense mixtures: at most this local packing
    rho *= f
    sp = [SimpleNamespace(d=float(d[i]), q=float(q[i]), rho_bulk=float(rb[i] * f), mu_el_bulk=0.0, mobile=True) for i in range(S)]
    sig = 0.5 * (d[:, None] + d[None, :])
    return SimpleNamespace(n=n, h=h, species=sp, T=300.0, terms=terms, eps_r=16.6, sw_eps=np.full((S, S), 0.1), sw_rout=sig + 0.3,
                           sw_gamma=1.2, sw_prefactor=0.5, precision=precision), rho


def one_electrolyte(case, seed):
    if case["kind"] != "equilibrium":
        return electrolyte(case["n"], case["S"], case["precision"], case.get("terms", ALL), seed)
    # plain Picard iteration converges for moderate coupling: a monovalent salt in water
    p, rho = electrolyte(case["n"], case["S"], case["precision"], HS | EC, seed, h=0.1, packing=0.1)
    p.eps_r = 78.5
    for i, s in enumerate(p.species):
        s.q = (-1.0) ** i
    return p, rho


def instances(case, seed):
    return [electrolyte(int(v), case["S"], case["precision"], ALL, seed * 1000 + k) for k, v in enumerate(case["sizes"].split(","))]


def quad_inputs(case, seed):
    """Fields of order one and one sphere radius each, 1.5 to 4 grid spacings."""
    r = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    f = 1 + torch.rand((case["F"], case["nx"], case["ny"], case["nz"]), generator=gen, device="cuda", dtype=torch.float64)
    return f, [0.05 * float(v) for v in np.linspace(1.5, 4.0, case["F"]) - r.uniform(0.0, 0.3, case["F"])]


_EV = None


def evaluator():
    """One evaluator for the process, as a program keeps it."""
    global _EV
    if _EV is None:
        _EV = pnp.Evaluator()
    return _EV


def prepare(case, seed):
    ev, kind = evaluator(), case["kind"]
    s = SimpleNamespace(case=case, ev=ev)
    if kind == "quad":
        s.f, s.radius = quad_inputs(case, seed)
        s.out = torch.empty((case["F"], 4) + tuple(s.f.shape[1:]), dtype=torch.float64, device="cuda")
        s.flags = (pnp.FLAG_CUBIC if case["cubic"] else 0) | (pnp.FLAG_APERIODIC if case["aperiodic"] else 0)
        return s
    if kind in ("batch", "plan"):
        s.problems, s.rhos = map(list, zip(*instances(case, seed)))
        s.ws = [torch.empty(ev.workspace_bytes(p), dtype=torch.uint8, device="cuda") for p in s.problems]
        s.mus, s.slots = ([torch.empty_like(r) for r in s.rhos] for _ in range(2))
        if kind == "plan":
            s.plan = ev.plan(s.problems, s.rhos, workspaces=s.ws, outs=s.mus, slots=s.slots)
        return s
    s.problem, s.rho = one_electrolyte(case, seed)
    if kind == "mu_ex":
        s.flags = pnp.FLAG_APERIODIC if case["aperiodic"] else 0
        s.mu = torch.empty(((3,) if case["per_term"] else ()) + tuple(s.rho.shape), dtype=torch.float64, device="cuda")
        s.slot = torch.empty_like(s.rho)
        s.ws = torch.empty(ev.workspace_bytes(s.problem, case["per_term"], flags=s.flags), dtype=torch.uint8, device="cuda")
    elif kind == "equilibrium":
        s.x = s.rho.clone()
    return s


def run(s):
    c, ev = s.case, s.ev
    kind = c["kind"]
    if kind == "mu_ex":
        out = list(ev.mu_ex(s.problem, s.rho, per_term=c["per_term"], out=s.mu, slot=s.slot, workspace=s.ws, flags=s.flags))
    elif kind == "batch":
        mus, slots, status = ev.batch(s.problems, s.rhos, workspaces=s.ws, outs=s.mus, slots=s.slots)
        out = [*mus, *slots, status]
    elif kind == "plan":
        s.plan.launch()
        out = [*s.mus, *s.slots, s.plan.status()]
    elif kind == "equilibrium":
        s.x.copy_(s.rho)
        mu, steps, res = ev.equilibrium(s.problem, s.x, lam=0.1, tol=0.0, max_iter=c["steps"])
        out = [s.x, mu, steps, res]
    elif kind == "quad":
        out = [ev.sphere_quadrature(s.f, s.radius, 0.05, order=c["order"], precision=c["precision"], flags=s.flags, out=s.out)]
    elif kind == "weighted":
        out = [ev.weighted_densities(s.problem, s.rho)]
    else:
        f, mu3 = ev.free_energy(s.problem, s.rho)
        out = [mu3, f]
    if c["precision"] == MIXED:
        out = [v.float() if isinstance(v, torch.Tensor) else v for v in out]
        if kind == "energy":
            out[1] = torch.tensor([f["hs"], f["el"], f["sh"], f["total"]], dtype=torch.float32)
    return out


# ---------------------------------------------------------------------------------------------------------------------
# bytes and operations of one pass

def _eval_work(n, S, outs, terms, extra=0):
    """rho in and `outs` arrays out; 3D real transforms of 2.5 N log2 N operations: the S densities, S results, and with a
    hard-sphere term the ten weighted densities and their ten derivatives; about 150 operations a point for the derivatives."""
    N = float(n) ** 3
    hs = bool(terms & (HS | WB))
    f = (2 * S + extra + (20 if hs else 0)) * 2.5 * N * math.log2(N) + (150 * N if hs else 0) + S * (S + 6) * 4 * N
    return 8.0 * S * N + 8.0 * outs * N, f


def work(case):
    kind = case["kind"]
    if kind == "quad":
        N = float(case["nx"]) * case["ny"] * case["nz"]
        # four weights on each offset of the merged stencil, about 4 pi r^2 times two cells of it (four for cubic)
        offs = sum(4 * math.pi * r * r * (4 if case["cubic"] else 2) for r in np.linspace(1.35, 3.85, case["F"]))
        return {"bytes": 40.0 * N * case["F"], "flops": 8.0 * offs * N}
    if kind in ("batch", "plan"):
        w = [_eval_work(int(v), case["S"], 2 * case["S"], ALL) for v in case["sizes"].split(",")]
        return {"bytes": sum(a for a, _ in w), "flops": sum(b for _, b in w)}
    n, S, terms = case["n"], case["S"], case.get("terms", ALL)
    if kind == "mu_ex":
        outs, extra = (4 * S if case["per_term"] else 2 * S), (2 * S if case["per_term"] else 0)
        b, f = _eval_work(n, S, outs, terms, extra)
        if case["aperiodic"]:  # the transforms are those of the doubled grid
            f = _eval_work(2 * n, S, outs, terms, extra)[1]
    elif kind == "equilibrium":
        b, f = (case["steps"] * v for v in _eval_work(n, S, 2 * S, HS | EC))
    elif kind == "weighted":
        b, f = _eval_work(n, S, 10, HS)
    else:
        b, f = _eval_work(n, S, 3 * S, terms, 2 * S)
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------------------------------------------------
# the same values in 64 bits, by torch FFTs

def _series(y, terms):
    y2, out, p = y * y, torch.zeros_like(y), torch.ones_like(y)
    for c in terms:
        out = out + c * p
        p = p * y2
    return out


def _j1x(y):
    """j1(y) / y."""
    z = y.clamp(min=0.5)
    s = [(-1) ** m / (math.factorial(2 * m + 1) * (2 * m + 3)) for m in range(9)]
    return torch.where(y < 0.5, _series(y, s), (torch.sin(z) - z * torch.cos(z)) / z ** 3)


def _rb(y):
    """int_0^1 t^2 sin(y t) / y dt: the transform of r theta(1 - r) over 4 pi."""
    z = y.clamp(min=1.0)
    s = [(-1) ** m / (math.factorial(2 * m + 1) * (2 * m + 4)) for m in range(12)]
    return torch.where(y < 1.0, _series(y, s), (2 * z * torch.sin(z) + (2 - z * z) * torch.cos(z) - 2) / z ** 4)


def _irb(y):
    """(1 - cos y) / y^2: the transform of theta(1 - r) / r over 4 pi."""
    return 0.5 * torch.sinc(y / (2 * math.pi)) ** 2


class _Space:
    """Wave-vectors of an n^3 grid of spacing h, in rfftn's layout."""

    def __init__(self, n, h):
        j = torch.fft.fftfreq(n, 1.0 / n, device="cuda", dtype=torch.float64)
        jz = torch.arange(n // 2 + 1, device="cuda", dtype=torch.float64)
        k0 = 2 * math.pi / (n * h)
        self.n = n
        self.k = k0 * torch.sqrt(j[:, None, None] ** 2 + j[None, :, None] ** 2 + jz[None, None, :] ** 2)
        s, sz = (k0 * torch.where(v.abs() == n / 2, torch.zeros_like(v), v) for v in (j, jz))  # odd functions vanish at the Nyquist index
        self.s = (s[:, None, None], s[None, :, None], sz[None, None, :])

    def fwd(self, a):
        return torch.fft.rfftn(a)

    def inv(self, a):
        return torch.fft.irfftn(a, s=(self.n,) * 3)

    def ball(self, a):
        return 4 * math.pi * a ** 3 * _j1x(self.k * a)


def _weighted(sp, rho, radii):
    """The ten weighted densities."""
    n = [0.0] * 4
    v1, v2 = 0.0, 0.0
    for R, r in zip(radii, rho):
        f = sp.fwd(r)
        shell, ball = f * torch.sinc(sp.k * R / math.pi), f * sp.ball(R)
        n = [n[0] + shell, n[1] + R * shell, n[2] + 4 * math.pi * R * R * shell, n[3] + ball]
        v1, v2 = v1 + ball / (4 * math.pi * R), v2 + ball  # the vector weights are gradients of the ball's
    return [sp.inv(a) for a in n] + [sp.inv(1j * s * v) for v in (v1, v2) for s in sp.s]


def _phi(n, wb):
    """(Phi_hs, its ten derivatives)."""
    n0, n1, n2, n3 = n[:4]
    v1, v2 = n[4:7], n[7:10]
    u = 1 - n3
    lu = torch.log1p(-n3)
    if wb:
        x = n3.clamp(min=0.05)
        ux, lx = 1 - x, torch.log1p(-x)
        g, dg = 1 / (x * ux ** 2) + lx / x ** 2, 2 / (x * ux ** 3) - 1 / (x * ux) ** 2 - 1 / (x * x * ux) - 2 * lx / x ** 3
        co = [(k + 1) * (k + 3) / (k + 2) for k in range(20)]
        gs = sum(c * n3 ** k for k, c in enumerate(co))
        dgs = sum(k * c * n3 ** (k - 1) for k, c in enumerate(co) if k)
        p, dp = (torch.where(n3 < 0.05, a, b) / (36 * math.pi) for a, b in ((gs, g), (dgs, dg)))
    else:
        p, dp = 1 / (24 * math.pi * u ** 2), 1 / (12 * math.pi * u ** 3)
    v12, v22 = (sum(a * b for a, b in zip(x, v2)) for x in (v1, v2))
    cube = n2 ** 3 - 3 * n2 * v22
    phi = -n0 * lu + (n1 * n2 - v12) / u + cube * p
    d = [-lu, n2 / u, n1 / u + 3 * (n2 * n2 - v22) * p, n0 / u + (n1 * n2 - v12) / u ** 2 + cube * dp]
    return phi, d + [-a / u for a in v2] + [-a / u - 6 * n2 * p * b for a, b in zip(v1, v2)]


def _terms(p, rho, aperiodic=False):
    """([hs, el, sh] each [S][N], sum of Phi_hs)."""
    m = p.n
    if aperiodic:
        rho = torch.nn.functional.pad(rho, (0, m) * 3)
    sp, S = _Space(rho.shape[-1], p.h), len(p.species)
    inside = (slice(0, m),) * 3
    radii = [0.5 * s.d for s in p.species]
    beta = 1.602176634e-19 / (1.380649e-23 * p.T)
    lb = 1.602176634e-19 / (4 * math.pi * 8.8541878128e-12) * 1e9 / p.eps_r * beta
    hs, el, sh = (torch.zeros((S, m, m, m), device="cuda", dtype=torch.float64) for _ in range(3))
    total = 0.0
    if p.terms & (HS | WB):
        w = _weighted(sp, rho, radii)
        if aperiodic:
            w = [torch.nn.functional.pad(a[inside], (0, m) * 3) for a in w]
        phi, d = _phi(w, bool(p.terms & WB))
        total = float(phi[inside].sum())
        d = [sp.fwd(a) for a in d]
        g1, g2 = (sum(1j * s * a for s, a in zip(sp.s, d[b:b + 3])) for b in (4, 7))
        for i, R in enumerate(radii):
            a = torch.sinc(sp.k * R / math.pi) * (d[0] + R * d[1] + 4 * math.pi * R * R * d[2])
            hs[i] = sp.inv(a + sp.ball(R) * (d[3] - g2 - g1 / (4 * math.pi * R)))[inside]
        del d, g1, g2, w
    kappa = math.sqrt(4 * math.pi * lb * sum(s.rho_bulk * s.q ** 2 for s in p.species))
    for j in range(S):
        f = sp.fwd(rho[j])
        dev = torch.zeros_like(rho[j])
        dev[inside] = rho[j][inside] - p.species[j].rho_bulk
        fd = sp.fwd(dev)
        for i in range(S):
            a, b = p.species[i], p.species[j]
            s = 0.5 * (a.d + b.d)
            if p.terms & EC:
                xi = kappa * s
                B = xi / (1 + xi + math.sqrt(1 + 2 * xi)) / s
                g = 2 * B * sp.ball(s) - 4 * math.pi * (B * B * s ** 4 * _rb(sp.k * s) + s * s * _irb(sp.k * s))
                el[i] += sp.inv(a.q * b.q * lb * g * fd)[inside]
            if p.terms & SW:
                sh[i] += sp.inv(-beta * p.sw_prefactor * p.sw_eps[i, j] * (sp.ball(p.sw_rout[i, j]) - sp.ball(s)) * f)[inside]
    return [hs, el, sh], total


def _exact_mu(p, rho, per_term=False, aperiodic=False):
    t = _terms(p, rho, aperiodic)[0]
    mu = t[0] + t[1] + t[2]
    return torch.stack(t) if per_term else mu, torch.exp(-mu)


def _exact_quad(case, f, radius):
    """The product rule node by node on the interpolant, the nodes' points merged by offset."""
    k, h, cubic = case["order"], 0.05, case["cubic"]
    x, w = np.polynomial.legendre.leggauss(k)
    out = []
    for fld, R in zip(f, radius):
        table = {}
        for i in range(k):
            th = 2 * math.pi * i / k
            for j in range(k):
                ph = 0.5 * math.pi * (x[j] + 1)
                nd = np.array([math.cos(th) * math.sin(ph), math.sin(th) * math.sin(ph), math.cos(ph)])
                W = R * R * math.sin(ph) * (2 * math.pi / k) * (0.5 * math.pi * w[j])
                pos = R / h * nd
                b = np.floor(pos).astype(int)
                t = pos - b
                if cubic:
                    ax = [[(-1, -v * (v - 1) * (v - 2) / 6), (0, (v + 1) * (v - 1) * (v - 2) / 2), (1, -(v + 1) * v * (v - 2) / 2),
                           (2, (v + 1) * v * (v - 1) / 6)] for v in t]
                else:
                    ax = [[(0, 1 - v), (1, v)] for v in t]
                for ox, wx in ax[0]:
                    for oy, wy in ax[1]:
                        for oz, wz in ax[2]:
                            key = (b[0] + ox, b[1] + oy, b[2] + oz)
                            table[key] = table.get(key, 0.0) + W * wx * wy * wz * np.array([1.0, *nd])
        H = max(max(abs(v) for v in key) for key in table)
        if case["aperiodic"]:
            g = torch.nn.functional.pad(fld, (H, H) * 3)
        else:
            g = fld
            for a, m in enumerate(fld.shape):
                g = g.index_select(a, torch.arange(-H, m + H, device="cuda") % m)
        acc = torch.zeros((4,) + tuple(fld.shape), device="cuda", dtype=torch.float64)
        for key, c in table.items():
            v = g[tuple(slice(H + o, H + o + m) for o, m in zip(key, fld.shape))]
            for q in range(4):
                acc[q] += float(c[q]) * v
        out.append(acc)
    return torch.stack(out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "quad":
        return [_exact_quad(case, *quad_inputs(case, seed))]
    if kind in ("batch", "plan"):
        e = [_exact_mu(p, r) for p, r in instances(case, seed)]
        return [a for a, _ in e] + [b for _, b in e] + [None]
    p, rho = one_electrolyte(case, seed)
    S = len(p.species)
    if kind == "mu_ex":
        return list(_exact_mu(p, rho, case["per_term"], case["aperiodic"]))
    if kind == "weighted":
        return [torch.stack(_weighted(_Space(p.n, p.h), rho, [0.5 * s.d for s in p.species]))]
    if kind == "equilibrium":
        rb = torch.tensor([s.rho_bulk for s in p.species], device="cuda", dtype=torch.float64)[:, None, None, None]
        bulk = SimpleNamespace(**{**vars(p), "n": 8})
        mb = sum(_terms(bulk, rb.expand(S, 8, 8, 8))[0])[:, :1, :1, :1]
        res = 0.0
        for _ in range(case["steps"]):
            mu = sum(_terms(p, rho)[0])
            new = 0.9 * rho + 0.1 * rb * torch.exp(mb - mu)
            res = float(((new - rho).abs() / rb).max())
            rho = new
        return [rho, mu, None, res]
    t, total = _terms(p, rho)
    h3 = p.h ** 3
    dev = rho - torch.tensor([s.rho_bulk for s in p.species], device="cuda", dtype=torch.float64)[:, None, None, None]
    e = {"hs": h3 * total, "el": 0.5 * h3 * float((dev * t[1]).sum()), "sh": h3 / (2 * p.sw_prefactor) * float((rho * t[2]).sum())}
    e["total"] = e["hs"] + e["el"] + e["sh"]
    if case["precision"] == MIXED:
        e = torch.tensor([e["hs"], e["el"], e["sh"], e["total"]], dtype=torch.float64)
    return [torch.stack(t), e]
