"""The x passes of more species than the streamed kernels take (mixed precision:
five and more from 128^3, four at 256^3) have elements per thread of their own:
the schedule bits of those passes, measured and tuned on the streamed kernels,
do not reach them."""
import pytest
import torch

import pnp_inputs as P
from paper_1407_0674_amd import MIXED, Evaluator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,S", [(128, 5), (192, 5), (256, 4), (256, 5)])
def test_one_schedule(n, S):
    gen = torch.Generator(device="cuda").manual_seed(5500 + n + S)
    prob, _ = P.many_species(8, S, 5500 + n + S, precision=MIXED)
    prob = prob.with_(n=n)
    rho = torch.rand((S, n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    for i, s in enumerate(prob.species):
        rho[i] = s.rho_bulk * (0.9 + 0.2 * rho[i])
    ev = Evaluator(0)
    try:
        first = None
        for bits in (0, 1 << 3, 1 << 7, 1 << 3 | 1 << 7):  # x forward, x back
            ev.tune_import(f"{MIXED} {n} s {bits}\n")
            mu, slot = ev.mu_ex(prob, rho)
            if first is None:
                first = mu.clone(), slot.clone()
            assert torch.equal(mu, first[0]) and torch.equal(slot, first[1]), bits
    finally:
        ev.close()
    del rho, mu, slot, first
    torch.cuda.empty_cache()
