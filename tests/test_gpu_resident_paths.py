"""Which launches a call takes, and what it does when a wait of a resident launch runs out
part way: the counts of the context say which path ran, and a wait bound of zero
from a chosen resident launch on makes that one give up.  The results equal those of ordinary
launches bit for bit wherever the repeat falls.
"""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2502_14589_amd import ch
from paper_2502_14589_amd.inputs import uniform_field


def say(msg):
    print(msg, flush=True)


def dev(y):
    import torch

    return torch.from_numpy(np.ascontiguousarray(y, dtype=np.float64)).to("cuda")


def problem(n, kind, prec=ch.CH_FP64):
    length = 64.0 if kind == "neumann" else 1.0
    bc = ch.CH_BC_NEUMANN if kind == "neumann" else ch.CH_BC_PERIODIC
    p = ch.Problem(2, n, 3.0 * length / n, precision=prec, bc=bc, length=length, mobility=(0.1, 1.0) if kind == "mobility" else None)
    return p, p.eps ** 2 * 64.0 * (n / length) ** 4


def call(c, what, p, rho, y0):
    """One call; its field, statistics and records.  Adaptive steps, restarted constant steps, LIM, the phi action."""
    y = dev(y0)
    if what == "ee":
        st, recs = c.run_ee(p, y, 400.0 / rho, max_steps=6, m_max=20, records=True)
    elif what == "constant":
        st, recs = c.run_ee(p, y, 60.0 / rho, max_steps=3, m_max=8, tol_phi_fixed=1e-6, constant_step=True, records=True)
    elif what == "lim":
        st, recs = c.run_lim(p, y, 600.0 / rho, max_steps=4, records=True)
    else:
        z = dev(y0)
        st, recs = c.phiv(p, y, z, 300.0 / rho, mode=ch.CH_PHI_RESTART if what == "phiv" else ch.CH_PHI_SHRINK, m_max=8), None
        y = z
    return y.cpu().numpy(), st, recs


CALLS = ["ee", "constant", "lim", "phiv", "shrink"]


@pytest.mark.parametrize("what", CALLS)
@pytest.mark.parametrize("n,kind,prec", [(13, "periodic", ch.CH_FP64), (96, "neumann", ch.CH_FP64), (125, "mobility", ch.CH_FP64),
                                         (96, "periodic", ch.CH_FP32_MIXED)])
def test_resident_against_ordinary_launches(n, kind, prec, what):
    """The counts tell the paths apart; the results do not."""
    say(f"paths of {what} n={n} {kind} prec={prec}")
    p, rho = problem(n, kind, prec)
    y0 = uniform_field(n, 2, 0.1, 0.4, seed=8800 + n)
    with ch.Context(0) as c, ch.Context(0) as o:
        o.set_resident(False)
        got, ref = call(c, what, p, rho, y0), call(o, what, p, rho, y0)
        info = c.resident_info()
        assert info["launches"] >= 1 and info["repeats"] == 0
        assert o.resident_info() == {"launches": 0, "repeats": 0, "paused_s": 0.0}
    assert got[1:] == ref[1:] and np.array_equal(got[0], ref[0])


# the launch that gives up: of adaptive steps the first, second (odd) and third (even); of constant
# steps and the phi action the first cycle, later cycles of a step and later steps
@pytest.mark.parametrize("what,after", [("ee", 0), ("ee", 1), ("ee", 2), ("ee", 5), ("constant", 0), ("constant", 1), ("constant", 2),
                                        ("constant", 5), ("constant", 7), ("lim", 0), ("lim", 1), ("lim", 2), ("phiv", 0),
                                        ("phiv", 1), ("phiv", 3), ("shrink", 0)])
@pytest.mark.parametrize("prec", [ch.CH_FP64, ch.CH_FP32_MIXED])
def test_repeat_from_a_later_launch(what, after, prec):
    say(f"repeat of {what} after {after} launches prec={prec}")
    n = 96
    p, rho = problem(n, "periodic", prec)
    y0 = uniform_field(n, 2, 0.1, 0.4, seed=8900)
    with ch.Context(0) as c, ch.Context(0) as o:
        o.set_resident(False)
        ref = call(o, what, p, rho, y0)
        c.set_resident(True, 0, after)
        got = call(c, what, p, rho, y0)
        info = c.resident_info()
        assert info["launches"] > after and info["repeats"] == 1
    assert got[1:] == ref[1:] and np.array_equal(got[0], ref[0])


@pytest.mark.parametrize("n", [96, 640])
def test_launches_of_several_streams_share_the_device(n):
    """Contexts of three threads, each on a stream of its own: at 96^2 their launches fit the device together, at 640^2
    some are refused the room and take the ordinary form.  No wait runs out, and all give the result of a run alone."""
    import torch

    say(f"three streams n={n}")
    p, rho = problem(n, "periodic")
    y0 = uniform_field(n, 2, 0.1, 0.4, seed=8950)
    with ch.Context(0) as o:
        o.set_resident(False)
        ref = [call(o, what, p, rho, y0) for what in ("ee", "lim")]
    got, infos, errors = [None] * 3, [None] * 3, []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                with ch.Context(0) as c:
                    for _ in range(8):
                        got[i] = [call(c, what, p, rho, y0) for what in ("ee", "lim")]
                        for g, r in zip(got[i], ref):
                            assert g[1:] == r[1:] and np.array_equal(g[0], r[0])
                    infos[i] = c.resident_info()
        except Exception as e:   # reported by the main thread
            errors.append(e)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
    assert sum(x["launches"] for x in infos) > 0 and sum(x["repeats"] for x in infos) == 0


@pytest.mark.parametrize("what", ["ee", "lim", "shrink"])
def test_an_expired_wait_is_remembered(what):
    """After a wait has run out the following calls take ordinary launches, until the pause is over; twice as long
    after the next one."""
    import time

    say(f"pause after an expired wait: {what}")
    p, rho = problem(96, "periodic")
    y0 = uniform_field(96, 2, 0.1, 0.4, seed=8960)
    with ch.Context(0) as c:
        call(c, what, p, rho, y0)   # workspaces
        n0 = c.resident_info()["launches"]
        c.set_resident(True, 0)
        call(c, what, p, rho, y0)
        first = c.resident_info()
        assert first["launches"] > n0 and first["repeats"] == 1 and 0.0 < first["paused_s"] <= 0.32
        call(c, what, p, rho, y0)
        second = c.resident_info()
        assert second["launches"] == first["launches"] and second["paused_s"] > 0.0
        time.sleep(second["paused_s"] + 0.01)
        call(c, what, p, rho, y0)
        third = c.resident_info()
        assert third["launches"] > first["launches"] and third["repeats"] == 2 and 0.32 < third["paused_s"] <= 0.64
        c.set_resident(True)
        call(c, what, p, rho, y0)
        assert c.resident_info()["repeats"] == 2 and c.resident_info()["launches"] > third["launches"]


def test_a_stream_with_a_cu_mask_takes_ordinary_launches():
    """Its CUs are fewer than the device's, and not known to be spread over the XCDs as the workgroups are."""
    import ctypes

    import torch

    say("stream with a CU mask")
    hip = ch.load_library()   # its HIP runtime
    stream = ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 8)(*[0xFFFFFFFF] * 4)
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), ctypes.c_uint32(8), mask) == 0
    p, rho = problem(96, "periodic")
    y0 = uniform_field(96, 2, 0.1, 0.4, seed=8970)
    with ch.Context(0) as o:
        o.set_resident(False)
        ref = [call(o, what, p, rho, y0) for what in ("ee", "lim")]
    s = torch.cuda.ExternalStream(stream.value)
    with torch.cuda.stream(s):
        with ch.Context(0) as c:
            got = [call(c, what, p, rho, y0) for what in ("ee", "lim")]
            assert c.resident_info()["launches"] == 0
    s.synchronize()
    for g, r in zip(got, ref):
        assert g[1:] == r[1:] and np.array_equal(g[0], r[0])


@pytest.mark.parametrize("steps", [1, 2, 5, 17, 40])
def test_lim_run_to_a_final_time_issues_few_steps_past_it(steps):
    """A run of a few steps to T does not issue many more that find it ended."""
    say(f"LIM to T in {steps} steps")
    p, rho = problem(64, "periodic")
    tau = 600.0 / rho
    y0 = uniform_field(64, 2, 0.1, 0.4, seed=8980)
    with ch.Context(0) as c, ch.Context(0) as o:
        o.set_resident(False)
        y, z = dev(y0), dev(y0)
        st, _ = c.run_lim(p, y, tau, T=(steps - 0.5) * tau)
        ref, _ = o.run_lim(p, z, tau, T=(steps - 0.5) * tau)
        assert st == ref and st["steps"] == steps and st["t"] == (steps - 0.5) * tau
        assert steps <= c.resident_info()["launches"] <= steps + 1
    assert np.array_equal(y.cpu().numpy(), z.cpu().numpy())


@pytest.mark.parametrize("n,prec", [(256, ch.CH_FP64), (1024, ch.CH_FP64), (1400, ch.CH_FP32_MIXED)])
def test_a_tuned_shape_keeps_the_resident_cycles(n, prec):
    """The tuner times ordinary launches; it does not keep a shape under which a run would have to take them."""
    say(f"tuned shape n={n} prec={prec}")
    p, rho = problem(n, "periodic", prec)
    with ch.Context(0) as c:
        c.tune_shape(p, m_max=30)
        c.run_ee(p, dev(uniform_field(n, 2, 0.1, 0.4, seed=8990)), 90.0 / rho, max_steps=1, m_max=30)
        assert c.resident_info()["launches"] == 1
