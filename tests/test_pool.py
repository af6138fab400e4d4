"""The pool of device and pinned host blocks without a GPU
(tests/sanitize/pool_checks.cpp: pool.cpp over HIP calls that keep count), under
AddressSanitizer + UndefinedBehaviorSanitizer and under ThreadSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("san", ["address,undefined", "thread"])
def test_pool(tmp_path, san):
    exe, d = str(tmp_path / "pool_checks"), os.path.join(ROOT, "tests", "sanitize")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=" + san, "-fno-sanitize-recover=all", "-Wall", "-Werror",
                    "-I", os.path.join(d, "fake_hip"), "-o", exe, os.path.join(d, "pool_checks.cpp"),
                    os.path.join(ROOT, "paper_2604_01050_amd", "csrc", "pool.cpp"), "-lpthread"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and "pool checks passed" in r.stdout, r.stdout + r.stderr[-2000:]
