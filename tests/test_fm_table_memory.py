"""The few-mismatch search's interval table is optional: memory that it cannot get is no error of the index.  The
build's allocation steps (paper_1402_4876_amd/csrc/fm_table.h) as host code, with failing allocations."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "_build", "sanitized")


def test_failed_allocations_mean_no_table():
    os.makedirs(BUILD, exist_ok=True)
    exe = os.path.join(BUILD, "fm_table")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", os.path.join(ROOT, "paper_1402_4876_amd", "csrc"),
                           os.path.join(ROOT, "tests", "fm_table_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1"))
    assert r.returncode == 0 and "table memory ok" in r.stdout, r.stdout + r.stderr[-3000:]
