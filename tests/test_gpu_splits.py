"""The per-vector contraction in splits of the Cholesky vectors (few walkers), with the 16-k chunks
past M left out, and with the walkers that the precision guard takes left to its FP64 pass:
N <= 16 and 16 < N <= 32 kernels at odd chunk counts, ranges of vectors that the splits do not
divide, one walker, an empty spin, several determinants.  Against the FP64 oracle (lockstep: the
traces of every vector drive the walk) and bitwise across walker counts, which change the splits."""

import numpy as np
import pytest

from oracle import afqmc as A
from synthetic import gen_system, noci_trial, random_walkers
from tests.parity_helpers import log, oracle_U_to_gpu, run_lockstep

pytestmark = pytest.mark.gpu

SHAPES = {
    # name: (M, N_up, N_dn, N_g, walkers)
    "m10": (10, 3, 2, 37, 3),
    "m40_one": (40, 11, 11, 133, 1),
    "m72": (72, 16, 9, 61, 6),
    "m100_dn0": (100, 12, 0, 90, 5),
    "n20_m44": (44, 20, 18, 131, 5),
    "n32_m112": (112, 32, 29, 75, 9),
    "n17_m24_g8": (24, 17, 16, 8, 4),
    "n35_m130": (130, 35, 0, 77, 3),
    "n50_m145": (145, 50, 49, 60, 2),
}


def _measure(s, U, nw, precision, tile=None, **kw):
    import torch

    import paper_1711_02242_amd as afq
    gs = afq.System.from_synthetic(s, dtau=0.005, precision=precision, **kw)
    if tile:
        gs.set_tile(tile)
    wk = gs.walkers(nw)
    gs.init(wk)
    wk.U.copy_(torch.from_numpy(oracle_U_to_gpu(U[0][:nw], U[1][:nw])))
    gs.measure(wk)
    torch.cuda.synchronize()
    return wk.e_loc.cpu().numpy()


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_split_lockstep(shape, precision):
    M, nu, nd, G, nw = SHAPES[shape]
    s = gen_system(M, nu, G, seed=71, n_dn=nd)
    log(f"splits {shape} {precision}")
    run_lockstep(s, nw, 4, dtau=0.005, precision=precision, rtol=1e-4,
                 label=f"splits-{shape}-{precision}", el_abs=1e-4)


def test_split_multidet():
    s = gen_system(40, 9, 150, seed=72)
    run_lockstep(s, 4, 4, dtau=0.005, precision="fp32", rtol=1e-4, label="splits-md",
                 trial=noci_trial(s, 3, seed=73))


@pytest.mark.parametrize("n,tile", [(12, None), (24, None), (12, "flat"), (21, "stack"),
                                    (21, "wide"), (35, None), (35, "stack"), (35, "flat")])
def test_results_do_not_depend_on_the_walker_count(n, tile):
    """Other walker counts take other splits: FP64 sums of the same FP32 terms."""
    s = gen_system(56, n, 211, seed=74)
    U = random_walkers(s, 700, seed=75, amplitude=0.4)
    ref = _measure(s, U, 700, "fp32", tile, theta_guard=np.inf)
    for nw in (1, 17, 130):
        e = _measure(s, U, nw, "fp32", tile, theta_guard=np.inf)
        assert np.abs(e - ref[:nw]).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("n", [14, 27])
def test_guard_takes_some_spins(n, precision):
    s = gen_system(60, n, 170, seed=76, n_dn=n - 1)
    nw = 70
    U = random_walkers(s, nw, seed=77, amplitude=1.0)
    U[1][1::3] += random_walkers(s, nw, seed=78, amplitude=2.5)[1][1::3]
    th = [np.array([np.abs(A.overlap_theta(p, u)[1]).max() for u in U[k]])
          for k, p in enumerate((s.phi_up, s.phi_dn))]
    cut = float(np.median(np.concatenate(th)))
    above = [t > cut for t in th]
    e64 = _measure(s, U, nw, "fp64")
    off = _measure(s, U, nw, precision, theta_guard=np.inf)
    some = _measure(s, U, nw, precision, theta_guard=cut)
    both, none = above[0] & above[1], ~(above[0] | above[1])
    log(f"guard N={n} {precision}: both {both.sum()}, none {none.sum()} of {nw}")
    assert both.any() and none.any()
    assert np.abs(some - e64)[both].max() <= 1e-10 * np.abs(e64).max()
    assert np.array_equal(some[none], off[none])
