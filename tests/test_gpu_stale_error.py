"""Reading statuses reports the status of the evaluation, not an error that some
other HIP call of the process had left for the next to find."""
import pytest
import torch

import pnp_inputs as P
from conftest import to_dev
from paper_1407_0674_amd import FLAG_ASYNC, MIXED, Evaluator

pytestmark = pytest.mark.gpu


def test_status_reads_after_a_foreign_error():
    prob, rho = P.many_species(16, 2, 5900, precision=MIXED)
    rd = to_dev(rho)
    ev = Evaluator(0)

    def fail():  # of an argument check on the host; the device is not reached
        assert ev.lib.hipSetDevice(9999) != 0
        return ev.lib.hipPeekAtLastError()

    try:
        plan = ev.plan([prob], [rd])
        plan.launch()
        ws = torch.empty(ev.workspace_bytes(prob), dtype=torch.uint8, device="cuda")
        ev.mu_ex(prob, rd, workspace=ws, flags=FLAG_ASYNC)
        torch.cuda.synchronize()
        if fail() == 0:
            pytest.skip("this runtime keeps no error")
        assert plan.status() == [0]
        fail()
        ev.read_status(ws)
        plan.close()
    finally:
        ev.lib.hipGetLastError()
        torch.cuda.synchronize()
        ev.close()
