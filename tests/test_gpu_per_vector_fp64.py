"""The FP64 contraction by products Omega^g, one per Cholesky vector, where the virtual-space form is
not used: few vectors against many amplitudes, or no virtual orbital (N = M).  In the FP64 mode (on
the matrix cores, and beyond their shapes on the vector units) and as the FP64 pass of the precision
guard, with every walker-spin above the threshold or only some; lockstep with the oracle, which the
traces of every vector drive."""

import ctypes as C
import math

import numpy as np
import pytest

from paper_1711_02242_amd import _lib as L
from synthetic import gen_system, noci_trial, random_walkers
from tests.parity_helpers import log, run_lockstep

pytestmark = pytest.mark.gpu

SHAPES = {
    # name: (M, N_up, N_dn, N_g)
    "n32_m128": (128, 32, 32, 20),
    "n31_m96_dn0": (96, 31, 0, 9),
    "n12_m100": (100, 12, 9, 5),
    "n_is_m": (6, 6, 6, 14),
    "n_is_m_up": (12, 12, 5, 30),
    "n20_is_m": (20, 20, 20, 33),
}
WIDE = {"n37_m150": (150, 37, 36, 11), "n40_is_m": (40, 40, 40, 9)}


def _per_vector(M, nu, nd, G):
    """The rule: no virtual orbital of an occupied spin, or fewer operations by Omega^g."""
    d = [n * (M - n) for n in (nu, nd) if n]
    return 0 in d or sum(2 * a * a + 4 * G * a for a in d) > 4 * G * M * (nu * nu + nd * nd)


@pytest.mark.parametrize("shape", list(SHAPES) + list(WIDE))
def test_fp64_mode(shape):
    M, nu, nd, G = {**SHAPES, **WIDE}[shape]
    assert _per_vector(M, nu, nd, G)
    s = gen_system(M, nu, G, seed=81, n_dn=nd)
    run_lockstep(s, 5, 4, dtau=0.005, U=random_walkers(s, 5, seed=82, amplitude=0.4), qr_period=3,
                 label=f"per-vector-{shape}")


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_guard_pass(shape, precision):
    M, nu, nd, G = SHAPES[shape]
    s = gen_system(M, nu, G, seed=83, n_dn=nd)
    U = random_walkers(s, 7, seed=84, amplitude=0.6)
    for guard in (1e-12, 0.7):
        run_lockstep(s, 7, 3, dtau=0.005, U=U, precision=precision, theta_guard=guard, rtol=1e-4,
                     el_abs=1e-4, label=f"per-vector-guard-{shape}-{precision}-{guard}")


def test_guarded_energies_are_fp64():
    import torch

    import paper_1711_02242_amd as afq
    from tests.parity_helpers import oracle_U_to_gpu
    s = gen_system(128, 32, 20, seed=85, n_dn=30)
    nw = 9
    U = random_walkers(s, nw, seed=86, amplitude=0.5)
    e = {}
    for prec, guard in (("fp64", None), ("fp32", 1e-12), ("bf16x3", 1e-12)):
        gs = afq.System.from_synthetic(s, dtau=0.005, precision=prec, theta_guard=guard)
        wk = gs.walkers(nw)
        gs.init(wk)
        wk.U.copy_(torch.from_numpy(oracle_U_to_gpu(*U)))
        gs.measure(wk)
        e[prec] = wk.e_loc.cpu().numpy()
    for prec in ("fp32", "bf16x3"):
        d = np.abs(e[prec] - e["fp64"]).max() / np.abs(e["fp64"]).max()
        log(f"per-vector guard {prec}: {d:.1e}")
        assert d <= 1e-12   # the same sums in the same kernel


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_multidet(precision):
    s = gen_system(64, 16, 4, seed=87, n_dn=15)
    assert _per_vector(64, 16, 15, 4)
    f64 = precision == "fp64"
    run_lockstep(s, 4, 4, dtau=0.005, precision=precision, rtol=1e-10 if f64 else 1e-4,
                 theta_guard=None if f64 else 1e-12, label=f"per-vector-md-{precision}",
                 trial=noci_trial(s, 4, seed=88))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", ["n32_m128", "n_is_m_up"])
def test_footprint(shape, precision):
    import paper_1711_02242_amd as afq
    M, nu, nd, G = SHAPES[shape]
    s = gen_system(M, nu, G, seed=89, n_dn=nd)
    gs = afq.System.from_synthetic(s, dtau=0.01, precision=precision)
    p = L.Params(M=M, n_up=nu, n_dn=nd, n_chol=G, dtau=0.01, e_trial=math.nan, n_taylor=6, qr_period=5,
                 pop_period=5, precision=L.PRECISIONS[precision], el_cap_C=2.0, w_max=math.nan,
                 fb_cap=1.0, flags=0, n_growth=0, theta_guard=math.nan)
    a, b, ws = C.c_size_t(), C.c_size_t(), C.c_size_t()
    L.check(gs.lib.afqmc_footprint_bytes(C.byref(p), 1, 33, C.byref(a), C.byref(b)), "footprint")
    L.check(gs.lib.afqmc_workspace_bytes(gs.handle, 33, C.byref(ws)), "workspace")
    nt = nu + nd
    assert a.value == gs.device_bytes
    assert b.value == ws.value + 256 + 33 * nt * M * 16 + 33 * (8 * 4 + 16 + 8)
