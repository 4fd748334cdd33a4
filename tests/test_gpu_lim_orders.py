"""The plan's node order where it changes hands: the lanes of one wave hold 2, 4, 8 or 16
nodes each (orders up to 128, 256, 512, 1024), the workgroup's threads more.  One LIM step
at the edges against the FP64 oracle, whose order it must take: the tolerance is that of the other
LIM steps (1e-10; other orders of the nodes lose many digits)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import ch_oracle as O
from paper_2502_14589_amd import ch
from paper_2502_14589_amd.inputs import uniform_field


@pytest.mark.parametrize("p", [3, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025])
def test_order_at_the_edges(p):
    import torch

    n, eps = 24, 0.1
    po = O.Problem(2, n, eps)
    y0 = uniform_field(n, 2, 0.3, 0.1, seed=9200)
    # eq. p: ceil((pi / 4) / (pi / 2 - atan(sqrt(tau lambda)))) = p in the middle of its interval
    tau = np.tan(np.pi / 2 - np.pi / 4 / (p - 0.5)) ** 2 / O.lambda_max(y0, po)
    y_ref, pr = O.lim_step(y0, po, tau)
    assert pr == p
    with ch.Context(0) as c:
        y = torch.from_numpy(y0.copy()).to("cuda")
        rec = c.step_lim(ch.Problem(2, n, eps), y, tau)
        assert rec["j"] == p
        d = y.cpu().numpy() - y_ref
        assert np.linalg.norm(d) <= 1e-10 * np.linalg.norm(y_ref)
