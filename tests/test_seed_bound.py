"""The bounds of the seeded bands (paper_1402_4876_amd/csrc/seed_bound.h, used by the band kernels and the runtime) as
host code against full tables: tests/seed_bound_check.cpp, built with UndefinedBehaviorSanitizer.  Random legal
scorings, and pairs built to sit at the edge of what a loss proves."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "_build", "sanitized")


@pytest.fixture(scope="module")
def check():
    os.makedirs(BUILD, exist_ok=True)
    exe = os.path.join(BUILD, "seed_bound.%d" % os.getpid())
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I",
                           os.path.join(ROOT, "paper_1402_4876_amd", "csrc"),
                           os.path.join(ROOT, "tests", "seed_bound_check.cpp"), "-o", exe])
    yield exe
    os.remove(exe)


@pytest.mark.parametrize("seed", [1, 2])
@pytest.mark.parametrize("mode", ["semiglobal", "local"])
def test_best_alignments_stay_inside_the_bounds(check, mode, seed):
    r = subprocess.run([check, mode, str(seed), "15000"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-2000:]
    assert "0 failures" in r.stdout
