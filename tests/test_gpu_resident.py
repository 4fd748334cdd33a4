"""Launches whose workgroups exchange data while they run, against the ordinary
launches of the same step.

Both form every point with the same expressions, so they agree bit for bit.
The ordinary launches are forced with a wait bound of zero
(CH_RESIDENT_WAIT_US, read when a context is created): the workgroups give up
at their first wait, exit, and the host repeats the step.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import ch_oracle as O
from paper_2502_14589_amd import ch
from paper_2502_14589_amd.inputs import uniform_field


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def dev(y):
    import torch

    return torch.from_numpy(np.ascontiguousarray(y, dtype=np.float64)).to("cuda")


@pytest.fixture(scope="module")
def ctx():
    c = ch.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def plain():
    """A context whose resident launches give up at once."""
    mp = pytest.MonkeyPatch()
    mp.setenv("CH_RESIDENT_WAIT_US", "0")
    c = ch.Context(0)
    mp.undo()
    yield c
    c.close()


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# one tile, tiles of the least size, one and two tiles per row, odd sides, many tiles
@pytest.mark.parametrize("n", [5, 13, 64, 97, 121, 250])
@pytest.mark.parametrize("kind", ["periodic", "neumann", "mobility", "eyre"])
def test_lim_stages(ctx, plain, n, kind):
    say(f"resident LIM n={n} {kind}")
    length = 64.0 if kind == "neumann" else 1.0
    h = length / n
    kw = {"eyre": kind == "eyre", "length": length}
    if kind == "mobility":
        kw["mobility"] = (0.1, 1.0)
    bc = ch.CH_BC_NEUMANN if kind == "neumann" else ch.CH_BC_PERIODIC
    p = ch.Problem(2, n, 3.0 * h, bc=bc, **kw)
    y0 = uniform_field(n, 2, 0.1, 0.4, seed=8100 + n)
    tau = 40.0 * h ** 4 / p.eps ** 2
    out = []
    for c in (ctx, plain):
        y = dev(y0)
        st, recs = c.run_lim(p, y, tau, max_steps=3, records=True)
        out.append((y.cpu().numpy(), st, recs))
    assert out[0][1:] == out[1][1:] and st["steps"] == 3 and recs[0]["j"] >= 10
    assert np.array_equal(out[0][0], out[1][0])
    if n <= 97:
        okw = {"eyre": kind == "eyre", "length": length, "mobility": kw.get("mobility")}
        po = O.Problem(2, n, 3.0 * h, bc="neumann" if kind == "neumann" else "periodic", **okw)
        y_ref, _ = O.lim_const_run(y0, po, tau, 3)
        assert rel(out[0][0], y_ref) <= 1e-10


def test_lim_run_to_a_final_time(ctx, plain):
    """The end of a run found on the device: adaptive steps until T, more than are issued between two looks."""
    n = 72
    p = ch.Problem(2, n, 0.04)
    y0 = uniform_field(n, 2, 0.1, 0.05, seed=8200)
    out = []
    for c in (ctx, plain):
        y = dev(y0)
        st, _ = c.run_lim(p, y, 1e-6, T=4e-4, tol=1e-4)
        out.append((y.cpu().numpy(), st))
    assert out[0][1] == out[1][1] and st["t"] == 4e-4 and st["steps"] > 32
    assert np.array_equal(out[0][0], out[1][0])


# one group; widths of 1, 2 and 4 columns per lane; a last strip of one column (FP64 strips are 124 wide, FP32 248);
# four, eight and twelve waves per workgroup (512 and 760 in FP64)
@pytest.mark.parametrize("prec", [ch.CH_FP64, ch.CH_FP32_MIXED])
@pytest.mark.parametrize("n,kind", [(5, "periodic"), (63, "periodic"), (64, "neumann"), (66, "mobility"), (125, "periodic"),
                                    (125, "neumann"), (249, "mobility"), (250, "neumann"), (512, "periodic"), (760, "periodic")])
def test_krylov_cycles(ctx, plain, n, kind, prec):
    """Adaptive steps (the first shortened by the trace, later ones converging early) and restarted cycles of a constant
    step: field, records and statistics equal those of the ordinary launches."""
    say(f"resident cycles n={n} {kind} prec={prec}")
    length = 64.0 if kind == "neumann" else 1.0
    h = length / n
    bc = ch.CH_BC_NEUMANN if kind == "neumann" else ch.CH_BC_PERIODIC
    p = ch.Problem(2, n, 3.0 * h, precision=prec, bc=bc, length=length, mobility=(0.1, 1.0) if kind == "mobility" else None)
    y0 = uniform_field(n, 2, 0.1, 0.4, seed=8400 + n)
    rho = p.eps ** 2 * 64.0 / h ** 4
    out = []
    for c in (ctx, plain):
        y = dev(y0)
        st, recs = c.run_ee(p, y, 400.0 / rho, max_steps=3, m_max=30, records=True)
        z = dev(y0)
        st2, recs2 = c.run_ee(p, z, 60.0 / rho, max_steps=2, m_max=8, tol_phi_fixed=1e-6, constant_step=True, records=True)
        out.append((y.cpu().numpy(), z.cpu().numpy(), st, recs, st2, recs2))
    assert out[0][2:] == out[1][2:] and st["steps"] == 3 and st2["steps"] == 2
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def test_phiv_cycles(ctx, plain):
    n = 96
    p = ch.Problem(2, n, 0.03)
    y0 = uniform_field(n, 2, 0.1, 0.4, seed=8500)
    out = []
    for c in (ctx, plain):
        y, z = dev(y0), dev(y0)
        rec = c.phiv(p, y, z, 2e-5, mode=ch.CH_PHI_RESTART, m_max=12)
        out.append((z.cpu().numpy(), rec))
    assert out[0][1] == out[1][1] and rec["cycles"] > 1
    assert np.array_equal(out[0][0], out[1][0])


def test_two_threads_share_the_device():
    """Three contexts in three threads at sizes that together exceed the device's CUs: some take the ordinary
    launches, all give the result of a run alone."""
    import threading

    n = 640
    p = ch.Problem(2, n, 0.01)
    y0 = uniform_field(n, 2, 0.1, 0.4, seed=8300)
    tau = 400.0 / n ** 4 / p.eps ** 2
    with ch.Context(0) as c:
        y = dev(y0)
        c.run_lim(p, y, tau, max_steps=4)
        c.run_ee(p, y, 1e-9, max_steps=3)
        ref = y.cpu().numpy()
    got = [None] * 3

    def work(i):
        with ch.Context(0) as c:
            y = dev(y0)
            for _ in range(5):
                y.copy_(dev(y0))
                c.run_lim(p, y, tau, max_steps=4)
                c.run_ee(p, y, 1e-9, max_steps=3)
            got[i] = y.cpu().numpy()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for g in got:
        assert np.array_equal(g, ref)


# two strips to a wave: widths of 1, 2 and 4 columns per lane, and a last workgroup partly or wholly filled
@pytest.mark.parametrize("n,kind,prec", [(701, "periodic", ch.CH_FP64), (699, "neumann", ch.CH_FP32_MIXED), (1000, "mobility", ch.CH_FP64),
                                         (1024, "periodic", ch.CH_FP64), (1054, "neumann", ch.CH_FP32_MIXED),
                                         (1300, "periodic", ch.CH_FP32_MIXED)])
def test_krylov_cycles_of_two_strips_per_wave(ctx, plain, n, kind, prec):
    test_krylov_cycles(ctx, plain, n, kind, prec)


@pytest.mark.parametrize("prec", [ch.CH_FP64, ch.CH_FP32_MIXED])
@pytest.mark.parametrize("m_max", [31, 32, 33, 47, 48])
def test_krylov_dimensions_across_the_test_orders(ctx, plain, m_max, prec):
    """Dimensions whose tests fill the smaller padded order, the larger one, and exceed it (ordinary launches)."""
    n = 90
    p = ch.Problem(2, n, 0.03, precision=prec)
    y0 = uniform_field(n, 2, 0.1, 0.4, seed=8700 + m_max)
    rho = p.eps ** 2 * 64.0 * n ** 4
    out = []
    for c in (ctx, plain):
        y = dev(y0)
        st, recs = c.run_ee(p, y, 0.7 * m_max * m_max / rho, max_steps=2, m_max=m_max, records=True)
        out.append((y.cpu().numpy(), st, recs))
    assert out[0][1:] == out[1][1:] and recs[0]["j"] >= min(m_max, 33)   # the larger ones converge before m_max
    assert np.array_equal(out[0][0], out[1][0])
