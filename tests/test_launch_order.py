"""The order of launches whose workgroups wait for each other, against a model
of a device (CPU, tests/sanitize/order_checks.cpp under AddressSanitizer and
UndefinedBehaviorSanitizer)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches_that_run_together_fit(tmp_path):
    exe = str(tmp_path / "order_checks")
    src = os.path.join(ROOT, "tests", "sanitize", "order_checks.cpp")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall",
                    "-Werror", "-o", exe, src], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "order checks passed" in r.stdout, r.stdout + r.stderr
