"""The CUs leased to resident launches (csrc/ch_lease.h), on the CPU: the launches that hold leases together fit
the device, XCD by XCD."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_14589_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <random>
#include <thread>
#include <vector>
#include "ch_lease.h"
constexpr int CUS = 256, XCDS = 8;
// CUs of the fullest XCD under launches whose workgroups go to the XCDs in turn, from the first on
static int fullest(const std::vector<int>& launches) {
    int most = 0;
    for (int x = 0; x < XCDS; ++x) {
        int n = 0;
        for (int c : launches) n += (c + XCDS - 1 - x) / XCDS;
        most = n > most ? n : most;
    }
    return most;
}
int main() {
    std::mt19937 rng(1);
    int worst = 0;
    for (int trial = 0; trial < 20000; ++trial) {
        std::vector<ResidentLease> l(12);
        std::vector<int> held;
        for (auto& x : l) {
            const int c = 1 + (int)(rng() % (trial % 2 ? 256 : 90));
            if (x.take(0, CUS, c)) held.push_back(c);
        }
        const int f = fullest(held);
        worst = f > worst ? f : worst;
    }
    std::printf("%d", worst);
    ResidentLease a, b, c, d, e;
    auto put = [](const char* sep, bool got) { std::printf("%s%d", sep, got); };
    put(" ", a.take(1, CUS, 81)), put("", b.take(1, CUS, 81)), put("", c.take(1, CUS, 81));
    a.release();
    put(" ", c.take(1, CUS, 81)), put("", d.take(1, CUS, 81));
    b.release(), c.release();
    put(" ", a.take(1, CUS, 256)), put("", d.take(1, CUS, 1)), put("", d.take(2, CUS, 1));
    put(" ", e.take(3, 0, 1)), put("", e.take(-1, CUS, 1)), put("", e.take(64, CUS, 1));
    std::printf("\n");
    // many threads: all given back in the end
    std::vector<std::thread> ts;
    for (int t = 0; t < 8; ++t)
        ts.emplace_back([t] {
            for (int i = 0; i < 20000; ++i) {
                ResidentLease l;
                l.take(4, CUS, 1 + (t * 31 + i * 7) % 256);
            }
        });
    for (auto& t : ts) t.join();
    ResidentLease all;
    std::printf("%d\n", all.take(4, CUS, 256));
}
"""


def test_leases_fit_every_xcd(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    (tmp_path / "lease.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(tmp_path / "lease.cpp"), "-o", str(tmp_path / "lease")],
                   check=True)
    out = subprocess.run([str(tmp_path / "lease")], capture_output=True, text=True, check=True).stdout.split()
    assert int(out[0]) <= 32            # the CUs of an XCD
    assert out[1:3] == ["110", "10"]    # 81 workgroups take 11 CUs of the first XCD: two launches fit beside each other, not three
    assert out[3] == "101" and out[4] == "000"
    assert out[5] == "1"
