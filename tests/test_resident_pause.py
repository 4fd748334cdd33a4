"""When resident launches are tried again after a wait ran out (csrc/ch_pause.h), on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_14589_amd", "csrc")

# calls of 0.3 ms; every resident launch of the first `bad` seconds waits its 0.1 s in vain
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "ch_pause.h"
int main(int, char** a) {
    const double bad = std::atof(a[1]), wait = 0.1, call = 3e-4, end = std::atof(a[2]);
    ResidentPause p;
    double now = 0.0, lost = 0.0, first_good = -1.0;
    int expiries = 0;
    while (now < end) {
        const bool resident = p.over(now);
        if (resident && now < bad) {
            now += wait;
            lost += wait;
            ++expiries;
            p.expired(now, wait);
        } else if (resident) {
            if (first_good < 0.0) first_good = now;
            p.passed();
        }
        now += call;
    }
    std::printf("%d %.6f %.6f %d\n", expiries, lost, first_good, p.level);
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("pause")
    (d / "pause.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "pause.cpp"), "-o", str(d / "pause")], check=True)

    def go(bad, end):
        out = subprocess.run([str(d / "pause"), str(bad), str(end)], capture_output=True, text=True, check=True).stdout.split()
        return int(out[0]), float(out[1]), float(out[2]), int(out[3])

    return go


def test_no_expiry_no_pause(run):
    assert run(0.0, 10.0) == (0, 0.0, 0.0, 0)


def test_pauses_grow_while_waits_run_out(run):
    """3.2 s, 6.4 s, 12.8 s ...: a share of the time that shrinks."""
    expiries, lost, _, _ = run(1e9, 100.0)
    assert expiries == 6 and lost < 0.01 * 100.0
    expiries, lost, _, _ = run(1e9, 3000.0)
    assert expiries == 10 and lost < 0.001 * 3000.0


def test_starts_over_once_launches_pass(run):
    expiries, _, first_good, level = run(5.0, 60.0)
    assert expiries == 2 and level == 0
    assert 3.4 + 6.4 <= first_good < 3.4 + 6.4 + 0.1
