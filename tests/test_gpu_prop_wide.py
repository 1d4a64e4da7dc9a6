"""The wide FP32 propagation (M > 128 or N_up + N_dn > 64) for every count of row blocks, with A in
registers and streamed, spins of different row-block counts, M at and past a multiple of 16:
lockstep with the FP64 oracle (shared fields) at the mixed-precision bars."""

import pytest

from synthetic import gen_system
from tests.parity_helpers import run_lockstep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n_up,n_dn", [
    (72, 40, 30), (128, 33, 32),                            # up to eight chunks of K: registers
    (130, 16, 15), (144, 17, 32), (145, 40, 3), (160, 48, 0),   # nine and ten: up to 48 orbitals
    (137, 49, 20), (161, 20, 16), (177, 64, 33), (224, 50, 64)])  # streamed
def test_wide_propagation(M, n_up, n_dn):
    s = gen_system(M, n_up, 12, seed=61, n_dn=n_dn)
    run_lockstep(s, 3, 2, dtau=0.005, precision="fp32", rtol=1e-4, el_abs=1e-4,
                 label=f"prop-{M}-{n_up}-{n_dn}")
