"""The rule by which a path that failed is tried again (csrc/backoff.h), compiled
by the host C++ compiler: what every use does when each try fails, when one
failure is followed by successes, and that no number of failures ends the tries."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1710_09178_amd", "csrc")

# argv: uses, and the tries that fail ("all" or a count of first ones); prints the uses that try, with their patience
PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "backoff.h"
int main(int, char** v) {
    stag::Backoff b;
    int fails = std::strcmp(v[2], "all") ? std::atoi(v[2]) : 1 << 30;
    for (int i = 0; i < std::atoi(v[1]); ++i) {
        if (!b.use()) continue;
        std::printf("%d %llu\\n", i, b.patience(3200));
        if (fails-- > 0) b.failed(); else b.worked();
    }
}
"""


@pytest.fixture(scope="module")
def tries(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("backoff")
    (d / "b.cpp").write_text(PROGRAM)
    r = subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "b.cpp"), "-o", str(d / "b")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(uses, fails):
        out = subprocess.run([str(d / "b"), str(uses), str(fails)], capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]

    return run


def test_one_failure_passes(tries):
    got = tries(40, 1)
    assert got[0] == (0, 3200)
    assert got[1] == (17, 100)  # the next 16 uses do without; the try has less patience
    assert got[2:] == [(i, 3200) for i in range(18, 40)]


def test_failures_thin_out_but_never_end_the_tries(tries):
    got = [i for i, _ in tries(20000, "all")]
    gaps = [b - a - 1 for a, b in zip(got, got[1:])]
    assert gaps[:7] == [16, 32, 64, 128, 256, 512, 1024] and set(gaps[6:]) == {1024}


def test_a_success_forgets_the_failures(tries):
    got = [i for i, _ in tries(400, 3)]
    assert got[:4] == [0, 17, 50, 115] and got[4:] == list(range(116, 400))
