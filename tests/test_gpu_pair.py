"""The contraction in the trial's virtual space (the default where it is used) against the FP64
oracle and against the per-vector kernels, at the edges of its tiles: d = N (M - N) amplitudes
just below, at and above multiples of 128 and of 16, one occupied or one virtual orbital, unequal
and empty spins, N_g around 128, walker counts around 64, non-orthonormal and multi-determinant
trials.  Static: E_L per walker.  Dynamic: lockstep runs, which the traces of every Cholesky
vector drive (a trace written to the wrong vector leaves sum_g t_g^2, hence E_L, unchanged)."""

import numpy as np
import pytest

from oracle import afqmc as A
from synthetic import config_system, diagonal_system, gen_system, noci_trial, random_walkers
from tests.parity_helpers import log, oracle_U_to_gpu, run_lockstep

pytestmark = pytest.mark.gpu

EL_ABS = {"fp64": None, "fp32": 1e-4, "bf16x3": 1e-4}   # Ha; FP64 relative 1e-10
SHAPES = {
    # name: (M, N_up, N_dn, N_g, walkers)
    "d12": (8, 2, 2, 32, 16),
    "d15_n_virtual_1": (6, 5, 3, 40, 3),
    "d127_n1": (128, 1, 1, 600, 2),
    "d128": (24, 8, 8, 127, 63),
    "d129_dn0": (46, 3, 0, 128, 65),
    "d144_d128": (25, 9, 8, 129, 64),
    "d256_d272": (33, 17, 16, 257, 5),
    "d1200": (60, 30, 28, 130, 130),
    "n33": (40, 33, 32, 200, 7),
    "n49_m70": (70, 49, 2, 500, 4),
    "m139": (139, 5, 5, 150, 4),
}


def _energies(s, U, nw, precision, tile=None, **kw):
    import torch

    import paper_1711_02242_amd as afq
    gs = afq.System.from_synthetic(s, dtau=0.005, precision=precision, **kw)
    if tile:
        gs.set_tile(tile)
    wk = gs.walkers(nw)
    gs.init(wk)
    wk.U.copy_(torch.from_numpy(oracle_U_to_gpu(*U)))
    gs.measure(wk)
    torch.cuda.synchronize()
    return wk.e_loc.cpu().numpy()


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_pair_static(shape, precision):
    M, nu, nd, G, nw = SHAPES[shape]
    s = gen_system(M, nu, G, seed=61, n_dn=nd)
    U = random_walkers(s, nw, seed=62, amplitude=0.5)
    S = A.setup(s.h0, s.h1, s.L, s.phi_up, s.phi_dn, 0.005)
    ref = A.init_walkers(S, nw, *U).e_loc
    e = _energies(s, U, nw, precision)
    d = np.abs(e - ref).max()
    log(f"pair static {shape} {precision}: max |dE_L| = {d:.2e} Ha")
    assert d < (EL_ABS[precision] or 1e-10 * np.abs(ref).max())
    if precision != "fp64":
        # the per-vector kernels on the same walkers
        assert np.abs(e - _energies(s, U, nw, precision, tile="flat")).max() < 1e-4


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", ["d15_n_virtual_1", "d129_dn0", "d144_d128", "n33"])
def test_pair_lockstep(shape, precision):
    M, nu, nd, G, nw = SHAPES[shape]
    s = gen_system(M, nu, G, seed=63, n_dn=nd)
    f64 = precision == "fp64"
    log(f"pair lockstep {shape} {precision}")
    run_lockstep(s, min(nw, 9), 6, dtau=0.005, precision=precision, rtol=1e-10 if f64 else 1e-4,
                 label=f"pair-{shape}-{precision}", **({} if f64 else dict(el_abs=1e-4)))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_pair_skew_trial(precision):
    """A trial with linearly independent but not orthonormal orbitals (Theorem 1.5)."""
    s = diagonal_system(20, 6, 90, seed=64, mix_trial=True)
    U = random_walkers(s, 70, seed=65, amplitude=0.4)
    S = A.setup(s.h0, s.h1, s.L, s.phi_up, s.phi_dn, 0.005)
    ref = A.init_walkers(S, 70, *U).e_loc
    d = np.abs(_energies(s, U, 70, precision) - ref).max()
    assert d < (EL_ABS[precision] or 1e-10 * np.abs(ref).max())


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_pair_multidet(precision):
    s = gen_system(26, 6, 140, seed=66, n_dn=5)
    trial = noci_trial(s, 5, seed=67)
    f64 = precision == "fp64"
    run_lockstep(s, 66 if f64 else 20, 5, dtau=0.005, precision=precision,
                 rtol=1e-10 if f64 else 1e-4, label=f"pair-md-{precision}", trial=trial)


@pytest.mark.parametrize("walkers", [1, 64, 150])
def test_pair_guard_lists(walkers):
    """Every walker-spin above the guard's threshold, none, and some of them: the ones above
    take the FP64 sums, the others keep theirs."""
    s = config_system("medium")
    U = random_walkers(s, walkers, seed=68, amplitude=1.0)
    U[0][::3] += random_walkers(s, walkers, seed=69, amplitude=2.5)[0][::3]
    e64 = _energies(s, U, walkers, "fp64")
    e_off = _energies(s, U, walkers, "fp32", theta_guard=np.inf)
    e_all = _energies(s, U, walkers, "fp32", theta_guard=1e-12)
    e_some = _energies(s, U, walkers, "fp32", theta_guard=1.0)
    assert np.abs(e_all - e64).max() <= 1e-10 * np.abs(e64).max()
    th = [np.array([np.abs(A.overlap_theta(p, u)[1]).max() for u in U[k]])
          for k, p in enumerate((s.phi_up, s.phi_dn))]
    above = [t > 1.0 for t in th]
    log(f"guard lists: {walkers} walkers, above 1.0: {above[0].sum()} up, {above[1].sum()} down")
    both, none = above[0] & above[1], ~(above[0] | above[1])
    assert np.abs(e_some - e64)[both].max(initial=0.0) <= 1e-10 * np.abs(e64).max()
    assert np.array_equal(e_some[none], e_off[none])
