"""The autotuner times the launches that calls make: below 192^3 the first pass
with the radial tables in it, not the two launches that pass timing splits them
into."""
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import pnp_inputs as P
from conftest import to_dev
from paper_1407_0674_amd import MIXED, Evaluator

pytestmark = pytest.mark.gpu


def _kernels(fn):
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    return {e.key for e in prof.key_averages()}


def test_first_pass_of_the_autotuner():
    prob, rho = P.many_species(32, 2, 5700, precision=MIXED)
    rd = to_dev(rho)
    ev = Evaluator(0)
    try:
        call = _kernels(lambda: ev.mu_ex(prob, rd))
        if not any("k_zfwd" in k for k in call):
            pytest.skip("the profiler sees no kernels here")
        tune = _kernels(lambda: ev.autotune([prob], [rd], reps=1))
    finally:
        ev.close()
    assert not any("k_tables" in k for k in call)
    assert not any("k_tables" in k for k in tune), sorted(k for k in tune if "k_tables" in k or "k_zfwd" in k)
