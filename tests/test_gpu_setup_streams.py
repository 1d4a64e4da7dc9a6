"""Setting a system up is a matter of its own stream: work of other streams is not waited for, and
what setup leaves queued on the stream is done before the first use of it."""

import numpy as np
import pytest

from oracle import afqmc as A
from synthetic import config_system, random_walkers
from tests.parity_helpers import log, oracle_U_to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_setup_does_not_wait_for_other_streams(precision):
    import torch

    import paper_1711_02242_amd as afq
    s = config_system("medium")
    nw = 6
    U = random_walkers(s, nw, seed=1, amplitude=0.4)
    S = A.setup(s.h0, s.h1, s.L, s.phi_up, s.phi_dn, 0.005)
    ref = A.init_walkers(S, nw, *U).e_loc
    Ug = torch.from_numpy(oracle_U_to_gpu(*U)).cuda()
    kw = dict(dtau=0.005, precision=precision, theta_guard=1e-12)   # every walker in FP64
    afq.System.from_synthetic(s, **kw).close()   # kernels loaded
    a = torch.ones((8192, 8192), device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    other, mine = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(other):
        for _ in range(300):   # about two seconds
            torch.mm(a, a, out=b)
        end = torch.cuda.Event()
        end.record()
    with torch.cuda.stream(mine):
        gs = afq.System.from_synthetic(s, **kw)
    waited = end.query()
    with torch.cuda.stream(mine):
        wk = gs.walkers(nw)
        gs.init(wk)
        wk.U.copy_(Ug)
        gs.measure(wk)
        mine.synchronize()
    e = wk.e_loc.cpu().numpy()
    torch.cuda.synchronize()
    d = np.abs(e - ref).max() / np.abs(ref).max()
    log(f"setup beside another stream's work ({precision}): dE {d:.1e}")
    assert not waited
    assert d < 1e-10


def test_guard_tables_of_a_small_system_cost_little():
    """The guard's tables of a tiny system are one allocation, one copy and four launches: setup
    with them takes at most 1.3 times as long as without (the fastest of many, in turn)."""
    import time

    import paper_1711_02242_amd as afq
    s = config_system("tiny")
    best = {}
    for i in range(120):
        for guard in (None, np.inf):
            t = time.perf_counter()
            gs = afq.System.from_synthetic(s, dtau=0.01, precision="fp32", theta_guard=guard)
            t = time.perf_counter() - t
            gs.close()
            if i >= 5:
                best[guard] = min(best.get(guard, t), t)
    log(f"setup {best[None] * 1e3:.3f} ms, without the guard {best[np.inf] * 1e3:.3f} ms")
    assert best[None] <= 1.3 * best[np.inf]


def test_guard_tables_of_many_determinants_cost_little():
    """No pool of host threads for each of many small determinants: setup of 1024 of them with the
    guard's tables takes at most 2.5 times as long as without (the fastest of a few, in turn)."""
    import time

    import paper_1711_02242_amd as afq
    from synthetic import gen_system
    s = gen_system(16, 4, 96, seed=7)
    rng = np.random.default_rng(8)
    nd = 1024
    ups, dns = (p + 0.1 * rng.standard_normal((nd, 16, 4)) for p in (s.phi_up, s.phi_dn))
    best = {}
    for i in range(5):
        for guard in (None, np.inf):
            t = time.perf_counter()
            gs = afq.System.multidet(s.h0, s.h1, s.L, np.ones(nd, dtype=complex), ups, dns, dtau=0.01,
                                     precision="fp32", theta_guard=guard)
            t = time.perf_counter() - t
            gs.close()
            best[guard] = min(best.get(guard, t), t)
    log(f"setup of {nd} determinants {best[None] * 1e3:.0f} ms, without the guard {best[np.inf] * 1e3:.0f}")
    assert best[None] <= 2.5 * best[np.inf]
