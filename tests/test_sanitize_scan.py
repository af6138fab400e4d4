"""Validation of dense couplings and the schedule table, which run on several
threads, under host sanitizers (CPU): tests/sanitize/scan_checks.cpp."""
import os
import subprocess

import pytest

from test_sanitize import ENV, ROOT


@pytest.mark.slow
@pytest.mark.parametrize("kind", ["asan", "tsan"])
def test_scan_and_schedule_under_sanitizers(kind):
    import importlib.util
    spec = importlib.util.spec_from_file_location("sbqa_build", os.path.join(ROOT, "paper_2604_01050_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    exe = mod.build_sanitized(kind, driver="scan_checks")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=dict(os.environ, **ENV[kind]))
    out = r.stdout + r.stderr
    assert r.returncode == 0 and "scan checks passed" in r.stdout, out[-4000:]
    assert "Sanitizer" not in out and "runtime error" not in out, out[-4000:]
