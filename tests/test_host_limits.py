"""The library's host side where the system refuses it threads or memory: an
error status, never an end of the process. Each check runs in a process of its
own whose address space is limited."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_CODE = """
import resource, sys
sys.path.insert(0, %r)
import numpy as np
import paper_2604_01050_amd as sb
import sbqa_instances as inst
what, spare = sys.argv[1], int(sys.argv[2])
if what == "schedule":      # Eq. 5 for 64 runs of 2000 steps
    E = inst.regular_graph(64, 3, 1)
    kw = dict(csr=inst.edges_to_csr(64, E, inst.gaussian_edges(len(E), 2)), R=8, runs=64, steps=2000)
elif what == "scan":        # a dense matrix of many row blocks
    kw = dict(J=inst.dense_gaussian(1500, 3), R=2, runs=2, steps=4)
else:                       # the schedule table alone is larger than the space left
    kw = dict(J=inst.sk_pm1(64, 4), R=2, runs=1000, steps=20000, jp_kind=sb.JP_LINEAR)
vm = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (vm + spare, vm + spare))
try:
    sb.sbqa_create(**kw)
    print("created")
except sb.SbqaError as e:
    print("status", e.status)
"""


# a thread needs 8 MB of address space for its stack
@pytest.mark.parametrize("what,spare,status", [("schedule", 4 << 20, -3), ("scan", 4 << 20, -3), ("table", 40 << 20, -2)])
def test_refused_threads_and_memory(what, spare, status):
    import torch
    r = subprocess.run([sys.executable, "-c", _CODE % ROOT, what, str(spare)], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    got = r.stdout.strip().splitlines()[-1]
    if status == -3 and torch.cuda.is_available():
        return              # creation goes on to the GPU there
    assert got == "status %d" % status, got
