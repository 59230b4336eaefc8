"""Four to six species at 192^3 and 256^3, whose x passes have forms of their own.

Splitting a species in two of the same kind leaves every potential as it was:
the benchmark's three-species electrolyte with one, two or three species split
is compared, everywhere and in both precisions, with the FP64 evaluation of the
three, which tests/test_gpu_fullsize.py holds to the oracle's samples at both
sizes.  FP64 within 1e-10 and mixed within 1e-5 of each term's largest magnitude
(the bars used there).  And the aperiodic mode's doubled 192^3 grid, per term,
against the oracle."""
import numpy as np
import pytest
import torch

import pnp_inputs as P
from conftest import relerr, to_dev
from oracle.aperiodic import mu_ex_aperiodic
from paper_1407_0674_amd import FLAG_APERIODIC, FP64, MIXED

pytestmark = pytest.mark.gpu

TOL = {FP64: 1e-10, MIXED: 1e-5}


@pytest.fixture(scope="module", params=[192, 256])
def three(request, ev):
    print(f"workload n={request.param}", flush=True)
    prob, rho = P.config3(n=request.param)
    rho = to_dev(rho)
    mu3, _ = ev.mu_ex(prob, rho, per_term=True, slotboom=False, precision=FP64)
    yield prob, rho, mu3.clone()
    del rho, mu3
    torch.cuda.empty_cache()


@pytest.mark.parametrize("S", [4, 5, 6])
def test_split_species(ev, three, S):
    prob, rho, want = three
    of = sorted(list(range(3)) + list(range(S - 3)))  # the kind of each species
    sp = []
    for i in of:
        s = prob.species[i]
        half = 0.5 if of.count(i) == 2 else 1.0
        sp.append(P.Species(s.d, s.q, s.rho_bulk * half, s.mu_el_bulk))
    grid = np.ix_(of, of)
    split = prob.with_(species=sp, sw_eps=np.asarray(prob.sw_eps)[grid], sw_rout=np.asarray(prob.sw_rout)[grid])
    r = torch.stack([rho[i] * (0.5 if of.count(i) == 2 else 1.0) for i in of])
    for precision in (FP64, MIXED):
        tol = TOL[precision]
        mu, slot = ev.mu_ex(split.with_(precision=precision), r)
        mu3, _ = ev.mu_ex(split.with_(precision=precision), r, per_term=True, slotboom=False)
        for k, i in enumerate(of):
            scale = [float(want[t, i].abs().max()) for t in range(3)]
            for t in range(3):
                assert float((mu3[t, k] - want[t, i]).abs().max()) <= tol * scale[t], (precision, t, k)
            total = want[:, i].sum(dim=0)
            assert float((mu[k] - total).abs().max()) <= tol * sum(scale), (precision, k)
            assert float((slot[k] * torch.exp(total) - 1.0).abs().max()) <= tol * sum(scale), (precision, k)
    del r, mu, slot, mu3, total
    torch.cuda.empty_cache()


def test_aperiodic_96_domain(ev):
    prob, rho = P.many_species(96, 2, 5800)
    print("oracle domain 96", flush=True)
    ref = mu_ex_aperiodic(prob, rho, "fft")
    rd = to_dev(rho)
    for precision in (FP64, MIXED):
        p = prob.with_(precision=precision)
        mu, _ = ev.mu_ex(p, rd, flags=FLAG_APERIODIC)
        mu3, _ = ev.mu_ex(p, rd, per_term=True, flags=FLAG_APERIODIC)
        mu, mu3 = mu.cpu().numpy(), mu3.cpu().numpy()
        for i in range(2):
            assert relerr(mu[i], ref["total"][i]) < TOL[precision], i
            for k, name in enumerate(("hs", "el", "sh")):
                assert relerr(mu3[k, i], ref[name][i]) < TOL[precision], (name, i)
    del rd
    torch.cuda.empty_cache()
