"""A batch (or autotune) with more requests of one size than the argument ring
holds is refused as a whole, and its requests' statuses say so."""
import pytest
import torch

import pnp_inputs as P
from conftest import to_dev

pytestmark = pytest.mark.gpu

ARG, NOMEM = -1, -3


def test_statuses_of_a_refused_list(ev):
    prob, rho = P.many_species(8, 1, 5600)
    other, rho16 = P.many_species(16, 2, 5601)
    rd, rd16 = to_dev(rho), to_dev(rho16)
    ws = torch.empty(ev.workspace_bytes(prob), dtype=torch.uint8, device="cuda")
    ws16 = torch.empty(ev.workspace_bytes(other), dtype=torch.uint8, device="cuda")
    mu, mu16 = torch.full_like(rd, 7.0), torch.full_like(rd16, 7.0)
    n = 2049
    reqs, keep, _, _ = ev._requests([prob] * n + [other, prob], [rd] * n + [rd16, rd], False, [ws] * n + [ws16, ws],
                                    [mu] * n + [mu16, mu], None)
    reqs[n + 1].T = -1.0  # refused for a reason of its own
    for call in (lambda: ev.lib.pnp_batch_mu_ex(ev.ctx, n + 2, reqs, ev._stream()),
                 lambda: ev.lib.pnp_autotune(ev.ctx, n + 2, reqs, 1, ev._stream())):
        assert call() == NOMEM
        torch.cuda.synchronize()
        assert [int(reqs[k].status) for k in range(n + 2)] == [NOMEM] * (n + 1) + [ARG]
        assert bool((mu == 7.0).all()) and bool((mu16 == 7.0).all())
