"""The modified Cholesky kernels compiled for the host and run with one thread per lane: the
vectors are the oracle's, and when a workgroup's wavefronts straddle the moment at which another
workgroup of the same launch records the end of the decomposition, no workgroup goes on (a pivot
from a mixture of old and new LDS contents would index the tensor out of range)."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle.mcd import modified_cholesky

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1711_02242_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("mcd") / "mcd_schedule")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-pthread", "-I", os.path.join(HERE, "host_hip"),
                    "-I", CSRC, "-o", exe, os.path.join(HERE, "host_hip", "mcd_schedule.cpp")],
                   check=True)
    return exe


@pytest.mark.parametrize("M,delta", [(9, 1e-2)])
def test_no_workgroup_goes_on_after_the_end(program, tmp_path, M, delta):
    rng = np.random.default_rng(M)
    B = rng.standard_normal((M, M, M))
    B = B + B.transpose(0, 2, 1)
    w = np.exp(-np.arange(M) / 1.5)
    eri = np.einsum("k,kpr,kqs->pqrs", w, B, B)
    Lo, _ = modified_cholesky(eri, delta)
    eri.tofile(tmp_path / "eri")
    r = subprocess.run([program, str(M), repr(delta), str(tmp_path / "eri"), str(tmp_path / "L")],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    L = np.fromfile(tmp_path / "L").reshape(-1, M, M)
    assert int(r.stdout) == len(L) == len(Lo)
    assert np.abs(L - Lo).max() < 1e-12 * np.abs(Lo).max()
