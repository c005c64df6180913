"""The tridiagonalisation by column launches: sizes that take it by themselves just above the
last-columns kernel, and sizes that take it only where resident launches cannot run (forced
with a launch that gives up).  Against LAPACK, with the tolerances of the resident reduction:
eigenvalues within 40 s u lambda_max, H within (1 - p/2) 100 40 s u sqrt(s) eps^(p/2-1)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")


@pytest.mark.parametrize("shape", [(4, 32, 128, 1, 97, 1), (4, 32, 64, 2, 55, 1), (4, 32, 32, 4, 10, 3), (4, 32, 32, 8, 16, 1),
                                   (4, 32, 32, 8, 17, 1), (4, 64, 64, 10, 10, 3), (4, 64, 64, 10, 15, 4), (6, 64, 64, 11, 20, 5)])
def test_column_launches(shape):
    T, P, Q, N1, N2, M = shape
    s = N1 * N2 * M
    say(f"column launches {shape} (s = {s})")
    rng = np.random.default_rng(s)
    x = (rng.standard_normal((T, P, Q)) + 1j * rng.standard_normal((T, P, Q))).astype(np.complex64)
    with slrx.Plan(P, Q, T, N1, N2, M, slrx.make_params(n_irls=1, n_cg=1)) as pl:
        pl.set_kspace(x)
        pl.set_mask(np.ones((T, P, Q), np.uint8))
        R = pl.step_gram()
        ref = np.linalg.eigvalsh(R)
        eps = 0.01 * ref[-1]
        slrx.lib().slrx_fault_stall(1)  # sizes of the resident reduction: the repeat takes column launches
        try:
            lam, H, _ = pl.step_weights(eps)
        finally:
            slrx.lib().slrx_fault_stall(0)
    tol = 40 * s * 2.0 ** -53
    assert np.all(np.diff(lam) >= 0)
    assert np.abs(lam - ref).max() <= tol * ref[-1]
    _, V, alpha = oracle.eig_weights(R, eps, 0.6)
    assert np.linalg.norm(H - oracle.weight_matrix(V, alpha)) <= 0.7 * 100 * tol * np.sqrt(s) * eps ** -0.7
