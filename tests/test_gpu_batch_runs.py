"""3-D FP64 batches, whose workgroups walk several of a grid's runs of planes one
after the other where the batch alone fills the device.  The sums are handed out run
by run, so every member is bit-equal to its run alone, whatever the group; and a
batch of many small grids, whose runs outnumber 32768, is taken."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2502_14589_amd import ch


def say(msg):
    print(msg, flush=True)


def fields(ns, seed):
    import torch

    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [torch.rand(n ** 3, device="cuda", dtype=torch.float64, generator=g) * 0.4 - 0.1 for n in ns]


def check(ctx, ns, members, method, seed):
    """Two steps of the batch and of `members` alone."""
    y0 = fields(ns, seed)
    ys = [y.clone() for y in y0]
    eps = [4.0 / n for n in ns]
    rho = [e * e * (12.0 * n * n) ** 2 for n, e in zip(ns, eps)]
    if method == "ee":
        _, rc = ctx.run_ee_batch(ys, ns, eps, dim=3, tau0=[40.0 / r for r in rho], max_steps=2, m_max=16, tol=1e-4)
    else:
        _, rc = ctx.run_lim_batch(ys, ns, eps, dim=3, tau0=[60.0 / r for r in rho], max_steps=2, tol=1e-3)
    assert rc == 0
    for i in members:
        y = y0[i].clone()
        p = ch.Problem(3, ns[i], eps[i])
        if method == "ee":
            ctx.run_ee(p, y, 40.0 / rho[i], max_steps=2, m_max=16, tol=1e-4)
        else:
            ctx.run_lim(p, y, 60.0 / rho[i], max_steps=2, tol=1e-3)
        assert np.array_equal(y.cpu().numpy(), ys[i].cpu().numpy()), (method, i, ns[i])


# 300 grids of 128 runs; 3640 of 24 runs, as many as the stencil tiles allow
@pytest.mark.parametrize("method", ["ee", "lim"])
@pytest.mark.parametrize("count,n", [(300, 32), (3640, 12)])
def test_many_small_grids(count, n, method):
    say(f"{method} batch of {count} x {n}^3")
    with ch.Context(0) as ctx:
        check(ctx, [n] * count, [0, 1, count // 2, count - 1], method, 9300)


# solo runs of 1, 1, 2, 2, 3, 4, 5 and 10 planes, the last of each partly filled or not; groups with a last
# one of fewer runs
@pytest.mark.parametrize("method", ["ee", "lim"])
def test_groups_of_runs(method):
    say(f"{method} batch of mixed 3-D grids")
    ns = [24, 33, 43, 64, 70, 97, 111, 160] + [32] * 40 + [5, 65]
    with ch.Context(0) as ctx:
        check(ctx, ns, list(range(8)) + [20, 48, 49], method, 9400)
