"""A batch that the host's memory cannot hold is refused with MDPE_ENOMEM, not with
the process's end (no GPU needed)."""
import subprocess
import sys

CODE = r"""
import resource, sys
import numpy as np
from paper_2101_10881_amd import mdpe
N = 200000
plan = mdpe.Plan(3, np.full(N, 2), np.tile([0, 1], N), 8, 2, device=-1)
vm = [int(l.split()[1]) for l in open("/proc/self/status") if l.startswith("VmSize")][0]
resource.setrlimit(resource.RLIMIT_AS, ((vm << 10) + (24 << 20),) * 2)
try:
    mdpe.Batch([plan] * 24)
    print("built")
except mdpe.MdpeError as e:
    print("refused", e.code == mdpe.MDPE_ENOMEM)
"""


def test_batch_beyond_memory():
    r = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-500:]
    assert r.stdout.split()[-2:] == ["refused", "True"]
