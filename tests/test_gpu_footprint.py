"""afqmc_footprint_bytes is host arithmetic: the process has opened no GPU after it (a server sizes
its jobs before it takes a device)."""

import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import os
from paper_1711_02242_amd.serve import JobSpec, footprint
for prec in ("fp64", "fp32", "bf16x3"):
    assert footprint(JobSpec(0, None, 64, 16, 16, 384, 512, 0, prec)) > 0
opened = [os.path.realpath("/proc/self/fd/" + f) for f in os.listdir("/proc/self/fd")]
assert not [p for p in opened if "kfd" in p or "/dri/" in p], opened
"""


def test_footprint_opens_no_gpu():
    subprocess.run([sys.executable, "-c", CODE], cwd=ROOT, check=True, timeout=100)
