"""Modified Cholesky on the GPU at the edges of its tiles: M^2 around the 64 elements a workgroup
takes, and more vectors than are staged in LDS at a time (1024).  The decomposition's own
property: every residual element is at most delta in modulus, no vector more than M (M + 1) / 2."""

import numpy as np
import pytest

from oracle.mcd import eri_matrix, modified_cholesky
from tests.parity_helpers import log
from tests.test_gpu_mcd import _eri

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,delta", [(1, 1e-8), (2, 1e-8), (8, 1e-7), (9, 1e-7), (16, 1e-6)])
def test_mcd_small_sizes_match_oracle(M, delta):
    import torch

    import paper_1711_02242_amd as afq
    eri = _eri(M, 70 + M, M * M)
    Lo, _ = modified_cholesky(eri, delta)
    Lg, conv = afq.modified_cholesky(torch.from_numpy(eri).cuda(), delta)
    Lg = Lg.cpu().numpy()
    log(f"mcd M={M}: {len(Lg)} vectors")
    assert conv and len(Lg) == len(Lo)
    assert np.abs(Lg - Lo).max() < 1e-10 * np.abs(Lo).max()


def test_mcd_more_vectors_than_staged():
    import torch

    import paper_1711_02242_amd as afq
    M, delta = 48, 1e-7
    rng = np.random.default_rng(5)
    B = rng.standard_normal((1600, M, M))
    B = (B + B.transpose(0, 2, 1)).reshape(1600, -1)
    V = (B.T @ B) / 1600.0
    eri = np.ascontiguousarray(V.reshape(M, M, M, M).transpose(0, 2, 1, 3))
    Lg, conv = afq.modified_cholesky(torch.from_numpy(eri).cuda(), delta)
    Lf = Lg.cpu().numpy().reshape(len(Lg), -1)
    log(f"mcd M={M}: {len(Lg)} vectors")
    assert conv and 1024 < len(Lg) <= M * (M + 1) // 2
    assert np.abs(eri_matrix(eri) - Lf.T @ Lf).max() <= delta * (1 + 1e-9) + 1e-11 * np.abs(V).max()
