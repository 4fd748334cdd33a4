"""Run lengths of the 3-D marching kernels and their groups in a batch (csrc/ch_runs.h), on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_14589_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "ch_runs.h"
int main() {
    for (int n = 5; n <= 420; ++n) {
        const int L = march_len(n, CH_FP64);
        std::printf("%d %d", n, L);
        for (long long planes : {march_planes(n), 3000LL, 9000LL, 1000000LL})
            for (int lim = 0; lim < 2; ++lim) {
                const int g = march_group(n, L, planes, lim);
                std::printf(" %d %d", g, march_groups(n, L, g));
            }
        std::printf("\n");
    }
    std::printf("set\n");
    for (int n = 5; n <= 420; ++n)
        for (int w : {1, 3, 8, 20, 64, 200, 700, 2048}) std::printf("%d %d %d %d\n", n, w, march_len(n, CH_FP64), march_len_set(n, CH_FP64, w));
}
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("runs")
    (d / "runs.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "runs.cpp"), "-o", str(d / "runs")], check=True)
    out = subprocess.run([str(d / "runs")], capture_output=True, text=True, check=True).stdout
    return [[[int(x) for x in line.split()] for line in part.splitlines()] for part in out.split("set\n")]


def ceil(a, b):
    return -(-a // b)


def test_groups_cover_every_run(rows):
    for n, L, *rest in rows[0]:
        nxy, runs = ceil(n, 64) * ceil(n, 8), ceil(n, L)
        assert 1 <= L <= 16
        for g, groups in zip(rest[::2], rest[1::2]):
            assert 1 <= g <= runs and groups == nxy * ceil(runs, g)   # the groups hold each run once
            assert g * L <= 16 or g == 1


def test_batches_that_runs_of_16_allow_stay_allowed(rows):
    """Members of built-in shape count by their stencil tiles (at most 2048): never fewer than their runs of 16 planes."""
    for n, *_ in rows[0]:
        tiles = min(ceil(n, 32) * ceil(n, 4) ** 2, 2048)
        assert min(ceil(n, 64) * ceil(n, 8) * ceil(n, 16), 2048) <= tiles


def test_runs_of_a_set_shape(rows):
    """Fewer workgroups than built in get longer runs, one each, and 16 planes where they have to loop over runs."""
    for n, w, built_in, L in rows[1]:
        items = lambda planes: ceil(n, 64) * ceil(n, 8) * ceil(n, planes)   # noqa: E731
        fits = [x for x in range(built_in, 17) if items(x) <= w]
        assert L == (fits[0] if fits else 16)
