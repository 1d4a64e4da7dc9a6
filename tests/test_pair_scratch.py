"""Workspace of the virtual-space contraction: the scratch of split traces holds what the schedule
asks for, for lists of any length, and a population's workspace grows by no more than Theta in FP64
(which the guard's FP64 pass reads) where the amplitudes and the scratch fit over the Taylor
buffers, and by tens of megabytes less than its largest size for a handful of walkers."""

import ctypes as C
import math
import os
import re
import shutil
import subprocess

import pytest

from paper_1711_02242_amd import _lib as L

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1711_02242_amd", "csrc")


def test_split_scratch_holds_the_schedule(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    text = open(os.path.join(CSRC, "contract_pair.hpp")).read()
    cut = lambda a, b: text[text.index(a):text.index(b, text.index(a))]  # noqa: E731
    (tmp_path / "pair_sizes.inc").write_text(
        "#include <stddef.h>\n#include <algorithm>\n#define __host__\n#define __device__\n"
        + cut("constexpr int PAIR_B", "inline void pair_free_tables")
        + cut("constexpr int PAIR_SPLIT", "struct PairArgs"))
    exe = str(tmp_path / "pair_scratch")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", str(tmp_path), "-o", exe,
                    os.path.join(HERE, "host_hip", "pair_scratch.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def _walker_bytes(M, N, G, nw, precision, guard=math.nan):
    p = L.Params(M=M, n_up=N, n_dn=N, n_chol=G, dtau=0.01, e_trial=math.nan, n_taylor=6, qr_period=5,
                 pop_period=5, precision=L.PRECISIONS[precision], el_cap_C=2.0, w_max=math.nan,
                 fb_cap=1.0, flags=0, n_growth=0, theta_guard=guard)
    a, b = C.c_size_t(), C.c_size_t()
    L.check(L.load().afqmc_footprint_bytes(C.byref(p), 1, nw, C.byref(a), C.byref(b)), "footprint")
    return b.value


@pytest.mark.parametrize("M,N,G", [(128, 32, 800), (64, 16, 384)])
@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
def test_guard_adds_theta_to_a_population(M, N, G, precision):
    nw = 1024
    more = _walker_bytes(M, N, G, nw, precision) - _walker_bytes(M, N, G, nw, precision, math.inf)
    theta = nw * 2 * N * M * 16
    assert theta <= more <= 1.02 * theta


def test_few_walkers_take_little_scratch():
    # 24 column tiles and splits of 64 walkers: the most that two column tiles are cut into
    few = _walker_bytes(128, 32, 800, 4, "fp64")
    assert few <= 3.9e6 + 28 * 64 * 800 * 16
