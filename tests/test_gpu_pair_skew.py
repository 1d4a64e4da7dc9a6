"""The FP64 contraction in the trial's virtual space with a trial far from orthonormal: V B in the
place of V, B invertible, gives the same local energies and force-bias traces (Theorem 1.5).  Each
is then a sum of terms whose rounding grows with cond(B), not with its square: tr Omega by a few
cond(B) units of rounding, at cond(B) = 1e6 1e-10 (a numpy model of both ways of forming the
tables has 5e-11, and 1e-5 through the inverse of V^T V)."""

import copy

import numpy as np
import pytest

from synthetic import gen_system, noci_trial, random_walkers
from tests.parity_helpers import log, oracle_U_to_gpu

pytestmark = pytest.mark.gpu


def _mix(n, cond, seed):
    rng = np.random.default_rng(seed)
    a, b = (np.linalg.qr(rng.standard_normal((n, n)))[0] for _ in range(2))
    return a @ np.diag(np.geomspace(1.0, 1.0 / cond, n)) @ b


def _measure(s, U, nw, precision, trial=None, **kw):
    """E_L, and U after one step with zero fields: y = -xbar = i sqrt(dtau) t."""
    import torch

    import paper_1711_02242_amd as afq
    kw = dict(dtau=0.01, precision=precision, qr_period=0, pop_period=0, **kw)
    if trial is None:
        gs = afq.System.from_synthetic(s, **kw)
    else:
        gs = afq.System.multidet(s.h0, s.h1, s.L, trial[0], np.array(trial[1]), np.array(trial[2]), **kw)
    wk = gs.walkers(nw)
    gs.init(wk)
    wk.U.copy_(torch.from_numpy(oracle_U_to_gpu(*U)))
    gs.measure(wk)
    e = wk.e_loc.cpu().numpy()
    gs.step(wk, seed=1, x=torch.zeros((nw, s.n_chol), dtype=torch.float64, device="cuda"))
    return e, wk.U.cpu().numpy()


@pytest.mark.parametrize("n_dn", [6, 0])
@pytest.mark.parametrize("cond", [1e3, 1e6])
def test_traces_and_energies_of_a_skew_trial(cond, n_dn):
    s = gen_system(24, 6, 90, seed=3, n_dn=n_dn)
    nw = 5
    U = random_walkers(s, nw, seed=5, amplitude=0.4)
    e0, U0 = _measure(s, U, nw, "fp64")
    k = copy.copy(s)
    k.phi_up = s.phi_up @ _mix(6, cond, 1)
    k.phi_dn = s.phi_dn @ _mix(n_dn, cond, 2)
    e, U1 = _measure(k, U, nw, "fp64")
    de, du = np.abs(e - e0).max() / np.abs(e0).max(), np.abs(U1 - U0).max() / np.abs(U0).max()
    log(f"skew trial cond {cond:.0e}: E_L {de:.1e}, U after a step {du:.1e}")
    # the traces' few units of rounding times cond; U takes dtau of them
    assert du <= 1e-15 * cond
    # the exchange multiplies two such matrices: 2.4e-19 cond^2 in the model
    assert de <= 1e-15 * cond + 2e-18 * cond ** 2


def test_later_determinants_skew_and_dependent():
    """The second determinant skew, the third with two equal columns (no overlap with a walker)."""
    s = gen_system(24, 6, 90, seed=3, n_dn=5)
    nw, cond = 5, 1e6
    U = random_walkers(s, nw, seed=5, amplitude=0.4)
    coeffs, ups, dns = noci_trial(s, 3, seed=7)
    B = [_mix(6, cond, 3), _mix(5, cond, 4)]
    twin = ups[2].copy()
    twin[:, 4] = twin[:, 1]
    flat = (np.array(coeffs), [ups[0], ups[1], twin], list(dns))
    skew = (np.array(coeffs), [ups[0], ups[1] @ B[0], twin], [dns[0], dns[1] @ B[1], dns[2]])
    skew[0][1] /= np.linalg.det(B[0]) * np.linalg.det(B[1])   # the same determinant
    e0, U0 = _measure(s, U, nw, "fp64", flat)
    e, U1 = _measure(s, U, nw, "fp64", skew)
    de, du = np.abs(e - e0).max() / np.abs(e0).max(), np.abs(U1 - U0).max() / np.abs(U0).max()
    log(f"skew determinant: E_L {de:.1e}, U after a step {du:.1e}")
    # r_1 carries the rounding of det T and det B too: N + N factors of relative error 2.2e-16 cond
    assert du <= 1e-14 * cond and de <= 1e-14 * cond + 2e-18 * cond ** 2
