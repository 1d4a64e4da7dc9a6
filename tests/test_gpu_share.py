"""The shared-row contraction kernel (FP32, N_g (N_up + N_dn) >= 49152): every count of wavefronts
per walker and of row tiles, odd and even N (an even block's last distance is half a pair set),
partial last groups, odd and even 16-k chunk counts, walker counts that leave slots of a workgroup
empty, lost walkers, an empty spin, the guard's list.  FP32 energies against the FP64 mode at the
mixed-precision bar of 1e-4 Ha, and those below the size where the kernel starts against those
above it."""

import numpy as np
import pytest

from synthetic import gen_system, random_walkers
from tests.parity_helpers import log, oracle_U_to_gpu

pytestmark = pytest.mark.gpu

EL_TOL = 1e-4   # Ha per walker

SHAPES = {
    # name: (M, N_up, N_dn, N_g, walkers)
    "n8_m130": (130, 8, 8, 3075, 11),      # one wavefront per walker, tiles of two blocks
    "n17_m150": (150, 17, 16, 1495, 4),
    "n31_m129": (129, 31, 32, 781, 3),
    "n33_m40": (40, 33, 33, 747, 1),       # three chunks of 16 k: two steps a group
    "n35_dn0": (60, 35, 0, 1407, 5),
    "n41_m72": (72, 41, 40, 607, 7),
    "n50_m64": (64, 50, 49, 499, 2),
    "n64_m100": (100, 64, 63, 389, 3),
    "n40_m224": (224, 40, 38, 631, 3),     # the most chunks
}


def _energies(s, U, nw, precision, lost=(), tile=None, **kw):
    import torch

    import paper_1711_02242_amd as afq
    gs = afq.System.from_synthetic(s, dtau=0.005, precision=precision, **kw)
    if tile:
        gs.set_tile(tile)
    wk = gs.walkers(nw)
    gs.init(wk)
    wk.U.copy_(torch.from_numpy(oracle_U_to_gpu(U[0][:nw], U[1][:nw])))
    for i in lost:
        wk.weight[i] = 0.0
    gs.measure(wk)
    torch.cuda.synchronize()
    return wk.e_loc.cpu().numpy()


@pytest.mark.parametrize("shape", list(SHAPES))
def test_energies_match_fp64(shape):
    M, nu, nd, G, nw = SHAPES[shape]
    assert G * (nu + nd) >= 49152
    s = gen_system(M, nu, G, seed=91, n_dn=nd)
    U = random_walkers(s, nw, seed=92, amplitude=0.3)
    ref = _energies(s, U, nw, "fp64")
    e = _energies(s, U, nw, "fp32", theta_guard=np.inf)
    log(f"share {shape}: |dE| {np.abs(e - ref).max():.2e} of {np.abs(ref).max():.1f}")
    assert np.abs(e - ref).max() <= EL_TOL


@pytest.mark.parametrize("tile", ["flat", "stack", "wide"])
def test_tiles_lost_and_guarded_walkers(tile):
    s = gen_system(100, 22, 1144, seed=93, n_dn=21)
    nw = 23
    U = random_walkers(s, nw, seed=94, amplitude=0.4)
    lost = (0, 5, 6, 7, 22)
    ref = _energies(s, U, nw, "fp64")
    e = _energies(s, U, nw, "fp32", lost=lost, tile=tile)
    some = _energies(s, U, nw, "fp32", lost=lost, tile=tile, theta_guard=1.0)
    live = np.setdiff1d(np.arange(nw), lost)
    assert np.abs(e - ref)[live].max() <= EL_TOL
    assert np.abs(some - ref)[live].max() <= EL_TOL
