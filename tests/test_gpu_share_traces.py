"""The shared-row contraction's traces, which the force bias of the next step is made of: steps in
lockstep with the oracle, and against the kernels it stands in for.  For the latter two systems that
differ in some last Cholesky vectors of zeros: one at N_g (N_up + N_dn) >= 49152, where the
shared-row kernel runs, one below, where the wide, flattened or stacked-row kernel does.  Traces are
the same chains of products and sums in all of them, so U is bitwise the same; the exchange's FP32
terms are grouped otherwise, 6e-8 / sqrt(4 N_g N) of E_L (1.2e-10 here), held to ten times that."""

import copy

import numpy as np
import pytest

from synthetic import gaussian_fields, gen_system, random_walkers
from tests.parity_helpers import log, oracle_U_to_gpu, run_lockstep

pytestmark = pytest.mark.gpu

SHAPES = {
    # name: (M, N_up, N_dn, N_g, walkers); N odd and even, a last group of 1 .. q - 1 blocks
    "n17_m150": (150, 17, 16, 1495, 4),
    "n33_m40": (40, 33, 33, 747, 1),
    "n35_dn0": (60, 35, 0, 1407, 5),
    "n41_m72": (72, 41, 40, 607, 7),
    "n64_m100": (100, 64, 63, 389, 3),
}


@pytest.mark.parametrize("shape", list(SHAPES))
def test_lockstep(shape):
    M, nu, nd, G, nw = SHAPES[shape]
    assert G * (nu + nd) >= 49152
    s = gen_system(M, nu, G, seed=95, n_dn=nd)
    run_lockstep(s, nw, 3, dtau=0.005, precision="fp32", rtol=1e-4, el_abs=1e-4,
                 U=random_walkers(s, nw, seed=96, amplitude=0.3), label=f"share-{shape}")


def test_lockstep_guarded():
    """N <= 32: the guard leaves some walker-spins of the tile's kernel to the FP64 pass."""
    s = gen_system(100, 22, 1144, seed=97, n_dn=21)
    assert 1144 * 43 >= 49152
    run_lockstep(s, 9, 3, dtau=0.005, precision="fp32", rtol=1e-4, el_abs=1e-4, tile="flat",
                 theta_guard=0.8, U=random_walkers(s, 9, seed=98, amplitude=0.5), label="share-guard")


@pytest.mark.parametrize("M,nu,nd,tile,nw", [(143, 35, 33, None, 5), (72, 41, 40, "stack", 40),
                                             (100, 22, 21, "flat", 11), (64, 50, 49, "wide", 130),
                                             (130, 8, 8, None, 3)])
def test_same_traces_as_the_kernels_it_stands_in_for(M, nu, nd, tile, nw):
    import torch

    import paper_1711_02242_amd as afq
    G = -(-49152 // (nu + nd))
    low = G - 3
    assert G * (nu + nd) >= 49152 > low * (nu + nd)
    s = gen_system(M, nu, G, seed=99, n_dn=nd)
    s.L[low:] = 0.0
    t = copy.copy(s)
    t.L, t.n_chol = s.L[:low].copy(), low
    U = random_walkers(s, nw, seed=100, amplitude=0.3)
    out = []
    for q in (s, t):
        gs = afq.System.from_synthetic(q, dtau=0.005, precision="fp32", theta_guard=np.inf)
        if tile:
            gs.set_tile(tile)
        wk = gs.walkers(nw)
        gs.init(wk)
        wk.U.copy_(torch.from_numpy(oracle_U_to_gpu(*U)))
        gs.measure(wk)
        e = [wk.e_loc.cpu().numpy()]
        for k in range(3):
            x = gaussian_fields(1, 0, np.arange(nw), k, G)[:, :q.n_chol]
            gs.step(wk, seed=1, x=torch.from_numpy(np.ascontiguousarray(x)).cuda())
            e.append(wk.e_loc.cpu().numpy())
        out.append((np.array(e), wk.U.cpu().numpy()))
    (e, Us), (f, Ut) = out
    d = np.abs(e - f).max() / np.abs(f).max()
    log(f"share against {tile or 'wide'} M={M} N={nu}+{nd}: E_L {d:.1e}, U {np.abs(Us - Ut).max():.1e}")
    assert np.array_equal(Us, Ut)
    assert d <= 1.2e-9
