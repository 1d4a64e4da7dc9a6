"""The end of a step on the GPU (weights, bounds and growth sums; one workgroup per walker, then
one over the population) against the oracle, at the edges of its loops: populations of one, of
one and several wavefronts, beyond 256 and 1024 walkers, and more field blocks than threads."""

import pytest

from synthetic import gen_system
from tests.parity_helpers import run_lockstep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw,n_chol,weight_mode", [
    (1, 9, "phaseless"), (64, 9, "phaseless"), (257, 9, "phaseless"), (1025, 9, "phaseless"),
    (1, 9, "hybrid"), (257, 9, "hybrid"), (3, 1030, "hybrid"), (3, 1030, "free")])
def test_end_of_step_follows_oracle(nw, n_chol, weight_mode):
    """Through a QR, a block end and a comb, the growth state included, at the FP64 bar."""
    s = gen_system(8, 2, n_chol, seed=5)
    run_lockstep(s, nw, 6, dtau=0.01, weight_mode=weight_mode,
                 mean_field=weight_mode != "phaseless", label=f"finish-{nw}-{n_chol}")
