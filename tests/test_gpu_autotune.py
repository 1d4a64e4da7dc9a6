"""The autotuner keeps what is fastest in the steps that follow: the time it returns is that of the
contraction's launch in a measurement, and no other variant is clearly faster there.  Few walkers
(the launch is split over the Cholesky vectors), more of them, and a size at which the shared-row
kernel stands in for three variants."""

import pytest

from paper_1711_02242_amd._lib import TILES
from synthetic import gen_system
from tests.parity_helpers import log

pytestmark = pytest.mark.gpu


def _launch_ms(gs, wk):
    best = float("inf")
    for _ in range(3):   # the best of three rounds: one hiccup of the host or the clock is not the kernel
        for _ in range(3):
            gs.measure(wk)
        gs.kernel_timing(True)
        for _ in range(8):
            gs.measure(wk)
        ms, n = gs.kernel_time(0)
        gs.kernel_timing(False)
        best = min(best, ms / n)
    return best


@pytest.mark.parametrize("M,N,G,nw", [(64, 16, 640, 8), (96, 23, 900, 128), (127, 31, 762, 214),
                                      (143, 35, 858, 60)])
def test_autotuned_tile_is_the_fastest_in_a_run(M, N, G, nw):
    import paper_1711_02242_amd as afq
    s = gen_system(M, N, G, seed=55)
    gs = afq.System.from_synthetic(s, dtau=0.005, precision="fp32")
    wk = gs.walkers(nw)
    gs.init(wk)
    tile, ms = min((gs.autotune(wk, reuse=False) for _ in range(3)), key=lambda r: r[1])
    gs.set_tile(tile)
    run = _launch_ms(gs, wk)
    others = {}
    for t in TILES:
        try:
            gs.set_tile(t)
        except RuntimeError:
            continue
        others[t] = _launch_ms(gs, wk)
    log(f"autotune M={M} N={N} W={nw}: {tile} {ms:.3f} ms, in a run {run:.3f}, "
        + " ".join(f"{t} {v:.3f}" for t, v in others.items()))
    assert abs(ms - run) <= 0.25 * run
    assert run <= 1.2 * min(others.values())
