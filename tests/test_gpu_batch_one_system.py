"""Several populations of one system in a batch: their steps run at the same time on branches of
the graph and add to the same counters of the rare-event bounds.  The counts are those of the
populations stepped one after the other."""

import pytest

from synthetic import config_system
from tests.parity_helpers import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32"])
def test_counters_of_populations_stepped_together(precision):
    import numpy as np

    import paper_1711_02242_amd as afq
    s = config_system("tiny")
    # sizes that end their steps at different offsets, some pairs of them together
    sizes, steps = (4, 16, 16, 40, 64, 64, 130, 200, 257), 300
    kw = dict(dtau=0.01, precision=precision, el_cap_C=0.02, theta_guard=1.0)

    def populations():
        gs = afq.System.from_synthetic(s, **kw)
        wks = [gs.walkers(nw) for nw in sizes]
        for wk in wks:
            gs.init(wk)
        gs.bound_counts(clear=True)
        return gs, wks

    gs, wks = populations()
    for i, wk in enumerate(wks):
        for _ in range(steps):
            gs.step(wk, seed=i)
    want, weights = gs.bound_counts(), [wk.weight.cpu().numpy() for wk in wks]
    gs, wks = populations()
    b = afq.Batch([(gs, wk) for wk in wks])
    for _ in range(steps):
        b.step(list(range(len(sizes))))
    got = gs.bound_counts()
    log(f"counters {precision}: {want}, together {got}")
    assert all(np.array_equal(a, wk.weight.cpu().numpy()) for a, wk in zip(weights, wks))
    assert want[0] > 0 and want[3] > 0
    assert got == want
    b.close()
