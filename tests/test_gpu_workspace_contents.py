"""Workspaces come to a call with whatever the memory held: outputs and statuses
do not depend on it.  Each entry point runs once in a workspace of zeros and once
in one of 0xff bytes (NaN in both precisions), bit for bit alike."""
import pytest
import torch

import pnp_inputs as P
from conftest import to_dev
from paper_1407_0674_amd import FLAG_APERIODIC, FP64, MIXED, Evaluator

pytestmark = pytest.mark.gpu


def _twice(call, nbytes):
    outs = []
    for byte in (0, 255):
        ws = torch.full((nbytes,), byte, dtype=torch.uint8, device="cuda")
        out = call(ws)
        outs.append([t.clone() for t in out])
        assert all(bool(torch.isfinite(t).all()) for t in outs[-1]), byte
    for a, b in zip(*outs):
        assert torch.equal(a, b)


# domains whose last row tiles reach past the domain's edge among them, under
# the default schedules and under each one alone
@pytest.mark.parametrize("precision", [FP64, MIXED])
@pytest.mark.parametrize("n,S", [(4, 2), (8, 3), (12, 1), (12, 5), (16, 2), (24, 3), (32, 4), (48, 2), (64, 1)])
def test_aperiodic(ev, n, S, precision):
    prob, rho = P.many_species(n, S, 5100 + 10 * n + S, precision=precision)
    rd = to_dev(rho)
    one, two = Evaluator(0), Evaluator(0)
    one.tune_import(f"{precision} {2 * n} s 0\n")
    two.tune_import(f"{precision} {2 * n} s {sum(1 << p for p in range(1, 10))}\n")
    try:
        for e in (ev, one, two):
            for per_term in (False, True):
                nb = e.workspace_bytes(prob, per_term, flags=FLAG_APERIODIC)
                _twice(lambda ws: e.mu_ex(prob, rd, per_term=per_term, workspace=ws, flags=FLAG_APERIODIC), nb)
    finally:
        one.close()
        two.close()


@pytest.mark.parametrize("precision", [FP64, MIXED])
@pytest.mark.parametrize("n,S", [(8, 3), (16, 5), (24, 2), (48, 4), (64, 3), (128, 2), (192, 1)])
def test_periodic(ev, n, S, precision):
    for terms in (P.TERMS_ALL, P.TERM_EC | P.TERM_SW):
        prob, rho = P.many_species(n, S, 5200 + 10 * n + S, precision=precision, terms=terms)
        rd = to_dev(rho)
        for per_term in (False, True):
            nb = ev.workspace_bytes(prob, per_term)
            _twice(lambda ws: ev.mu_ex(prob, rd, per_term=per_term, workspace=ws), nb)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [8, 24, 64])
def test_other_entries(n):
    prob, rho = P.many_species(n, 2, 5300 + n, terms=P.TERMS_ALL, precision=FP64)
    rd = to_dev(rho)
    e = Evaluator(0)

    def with_ws(ws, fn):
        e._ws = {"default": ws}
        return fn()

    def energy():
        f, mu3 = e.free_energy(prob, rd)
        return mu3, torch.tensor([f[k] for k in ("hs", "el", "sh", "total")])

    def equilibrium():
        x = rd.clone()
        mu, it, res = e.equilibrium(prob, x, lam=0.05, tol=0.0, max_iter=3)
        return x, mu, torch.tensor([float(it), res])

    try:
        nb = e.workspace_bytes(prob, True)
        _twice(lambda ws: with_ws(ws, energy), nb)
        _twice(lambda ws: with_ws(ws, equilibrium), nb)
        _twice(lambda ws: with_ws(ws, lambda: (e.weighted_densities(prob, rd),)), nb)
        _twice(lambda ws: e.batch([prob], [rd], workspaces=[ws])[0], nb)
    finally:
        e._ws = {}
        e.close()


# the bytes asked for are those of the arrays that the passes use
@pytest.mark.parametrize("n,S", [(16, 1), (48, 8), (64, 5)])
def test_size(ev, n, S):
    prob, _ = P.many_species(8, S, 5400 + S, precision=FP64, terms=P.TERM_HS)
    h, m = n // 2, 3 * (n // 2) ** 2 + 1
    spectra = (2 * S + 10) * (n * n * h + n * n) * 16
    need = 256 + (n * n + 2 * 1024 + 4) * 8 + m * S * 16 + spectra
    assert need <= ev.workspace_bytes(prob.with_(n=n)) <= need + 8 * 256
