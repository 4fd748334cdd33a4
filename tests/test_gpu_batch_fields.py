"""How a batch takes its fields in and gives them back: one launch for four or more
members whose fields lie apart in the device's memory (16-byte or single values by
alignment, odd counts), a copy per member otherwise.  Every member is bit-equal to its run
alone, and nothing beside the fields is written."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2502_14589_amd import ch
from paper_2502_14589_amd.inputs import uniform_field


@pytest.mark.parametrize("method", ["ee", "lim"])
@pytest.mark.parametrize("ns,shift", [([8, 9, 33], 0), ([8, 9, 33, 64], 0), ([8, 9, 33, 65], 1), ([5] * 9 + [130], 1)])
def test_fields_of_a_batch(ns, shift, method):
    import torch

    with ch.Context(0) as ctx:
        total = sum(n * n + 3 for n in ns) + 8
        pool = torch.full((total,), 7.0, dtype=torch.float64, device="cuda")
        fields, solo, at = [], [], shift
        used = torch.zeros(total, dtype=torch.bool)
        for i, n in enumerate(ns):
            y0 = torch.from_numpy(uniform_field(n, 2, 0.1, 0.3, seed=9000 + i).reshape(-1).copy())
            f = pool[at:at + n * n]
            f.copy_(y0)
            used[at:at + n * n] = True
            fields.append(f)
            solo.append(y0.to("cuda"))
            at += n * n + (3 if i % 2 else 2)
        if method == "ee":
            _, rc = ctx.run_ee_batch(fields, ns, [0.1] * len(ns), tau0=1e-5, max_steps=2, m_max=10, tol=1e-4)
        else:
            _, rc = ctx.run_lim_batch(fields, ns, [0.1] * len(ns), tau0=1e-6, max_steps=2, tol=1e-3)
        assert rc == 0
        for i, n in enumerate(ns):
            p = ch.Problem(2, n, 0.1)
            if method == "ee":
                ctx.run_ee(p, solo[i], 1e-5, max_steps=2, m_max=10, tol=1e-4)
            else:
                ctx.run_lim(p, solo[i], 1e-6, max_steps=2, tol=1e-3)
            assert np.array_equal(solo[i].cpu().numpy(), fields[i].cpu().numpy()), (i, n)
        assert bool((pool.cpu()[~used] == 7.0).all())


def test_members_that_share_a_field():
    """The last member's result stands, as with a copy each."""
    import torch

    with ch.Context(0) as ctx:
        y0 = torch.from_numpy(uniform_field(16, 2, 0.1, 0.3, seed=9100).reshape(-1).copy()).to("cuda")
        y, z = y0.clone(), y0.clone()
        ctx.run_ee_batch([y] * 5, [16] * 5, [0.1] * 5, tau0=[1e-5] * 4 + [2e-5], max_steps=2, m_max=10, tol=1e-4)
        ctx.run_ee(ch.Problem(2, 16, 0.1), z, 2e-5, max_steps=2, m_max=10, tol=1e-4)
        assert np.array_equal(y.cpu().numpy(), z.cpu().numpy())
