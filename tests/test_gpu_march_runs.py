"""FP64 run lengths of the z-marching kernels (the planes a workgroup walks),
which the host picks per grid: 1 (42^3), 2 (43^3, a last run of one plane),
3 (70^3, likewise), 5 (111^3, likewise), 10 (160^3, no remainder).

Against the FP64 oracle: one EE2 step with a residual-time trace's iterations
(matvec and estimate pass) and one LIM step with its estimate, fields to 1e-10
in relative L2 and max-abs, as everywhere for FP64 steps of these lengths.  A
batch of grids with different lengths is bit-equal to its solo runs.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import ch_oracle as O
from paper_2502_14589_amd import ch
from paper_2502_14589_amd.inputs import uniform_field


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available()
    c = ch.Context(0)
    yield c
    c.close()


def dev(y):
    import torch

    return torch.from_numpy(np.ascontiguousarray(y, dtype=np.float64)).to("cuda")


def close(y, y_ref):
    d = y.cpu().numpy() - y_ref
    assert np.linalg.norm(d) <= 1e-10 * np.linalg.norm(y_ref) and np.max(np.abs(d)) <= 1e-10 * np.max(np.abs(y_ref))


@pytest.mark.parametrize("n", [42, 43, 70, 111, 160])
def test_run_lengths(ctx, n):
    eps = 4.0 / n
    po, pg = O.Problem(3, n, eps), ch.Problem(3, n, eps)
    rho = eps ** 2 * (12.0 * n * n) ** 2
    y0 = uniform_field(n, 3, 0.1, 0.3, seed=8500 + n)
    tau = 40.0 / rho
    y_ref, tau_ref, info = O.ee_step(y0, po, tau, 1e-8, 20)
    y = dev(y0)
    rec = ctx.step_ee(pg, y, tau, m_max=20, tol_phi_fixed=1e-8)
    assert rec["j"] == info.j
    close(y, y_ref)
    tau = 60.0 / rho
    y_ref, p = O.lim_step(y0, po, tau)
    y = dev(y0)
    rec = ctx.step_lim(pg, y, tau, tol=1e-2)
    assert rec["j"] == p
    close(y, y_ref)


def test_batch_of_run_lengths_equals_solo(ctx):
    ns = [43, 24, 70, 97, 111]
    y0 = [uniform_field(n, 3, 0.1, 0.1, seed=8600 + n) for n in ns]
    for method in ("ee", "lim"):
        f = [dev(y) for y in y0]
        if method == "ee":
            _, rc = ctx.run_ee_batch(f, ns, [0.05] * len(ns), dim=3, tau0=1e-4, max_steps=2, m_max=20, tol=1e-4)
        else:
            _, rc = ctx.run_lim_batch(f, ns, [0.05] * len(ns), dim=3, tau0=1e-6, max_steps=2, tol=1e-3)
        assert rc == 0
        for i, n in enumerate(ns):
            y = dev(y0[i])
            if method == "ee":
                ctx.run_ee(ch.Problem(3, n, 0.05), y, 1e-4, max_steps=2, m_max=20, tol=1e-4)
            else:
                ctx.run_lim(ch.Problem(3, n, 0.05), y, 1e-6, max_steps=2, tol=1e-3)
            assert np.array_equal(y.cpu().numpy(), f[i].cpu().numpy()), (method, n)
