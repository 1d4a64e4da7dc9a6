"""The counters of the rare-event bounds belong to the system, whose populations a batch steps at
the same time: k_step_finish, compiled for the host, of three populations that all read the
counters before any of them has written.  Nothing that one of them counted is lost."""

import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1711_02242_amd", "csrc")


def test_populations_finishing_together_lose_no_count(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    text = open(os.path.join(CSRC, "kernels_fp64.hpp")).read()
    kernel = re.search(r"^__global__ [^;{]*\bk_step_finish\(.*?^}\n", text, re.S | re.M).group(0)
    (tmp_path / "k_step_finish.inc").write_text(kernel)
    exe = str(tmp_path / "together")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-pthread", "-I", os.path.join(HERE, "host_hip"),
                    "-I", CSRC, "-I", str(tmp_path), "-o", exe,
                    os.path.join(HERE, "host_hip", "step_finish_together.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60, check=True).stdout
    # capped energies, capped weights, force-bias caps, live walkers, guarded walkers
    assert [int(v) for v in out.split()] == [100 + 3, 200 + 6, 300, 400 + 4 + 299 + 63, 500]
