"""The eigen-decomposition chain at the Gram sizes where its kernels change shape, in FP64:
eigenvalues and H of a weights step against LAPACK's of the Gram matrix the same plan
returns.

Tolerances: Householder reduction, divide and conquer and back-transformation are backward
stable, so the eigenpairs are those of R + dR with ||dR|| <= c(s) u ||R||, u = 2^-53; the
errors grow about linearly with s and c(s) = 40 s bounds both sides together.  An eigenvalue
then moves by at most ||dR||, and H = (R + eps)^(p/2-1) by (1 - p/2) eps^(p/2-2) ||dR||,
(1 - p/2) (lambda_max / eps) c(s) u relative to ||H||_2 = eps^(p/2-1) at most (||.||_F over
||.||_2 gives another sqrt(s) at most)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")

U = 2.0 ** -53


def check(shape, rank_deficient=False):
    T, P, Q, N1, N2, M = shape
    s = N1 * N2 * M
    rng = np.random.default_rng(s)
    x = (rng.standard_normal((T, P, Q)) + 1j * rng.standard_normal((T, P, Q))).astype(np.complex64)
    if rank_deficient:  # one smooth image in every frame: most eigenvalues at round-off
        img = np.exp(-((np.arange(P)[:, None] - P / 2) ** 2 + (np.arange(Q)[None] - Q / 2) ** 2) / (P * Q / 16))
        x = np.repeat(np.fft.fft2(img, norm="ortho")[None], T, 0).astype(np.complex64)
    with slrx.Plan(P, Q, T, N1, N2, M, slrx.make_params(n_irls=1, n_cg=1)) as pl:
        pl.set_kspace(x)
        pl.set_mask(np.ones((T, P, Q), np.uint8))
        R = pl.step_gram()
        ref = np.linalg.eigvalsh(R)
        eps = 0.01 * ref[-1]
        lam, H, _ = pl.step_weights(eps)
    tol = 40 * s * U
    assert np.all(np.diff(lam) >= 0)
    assert np.abs(lam - ref).max() <= tol * ref[-1]
    ev, V, alpha = oracle.eig_weights(R, eps, 0.6)
    H_ref = oracle.weight_matrix(V, alpha)
    assert np.linalg.norm(H - H_ref) <= 0.7 * 100 * tol * np.sqrt(s) * eps ** -0.7


@pytest.mark.parametrize("shape", [(2, 32, 32, 1, 1, 1), (2, 32, 32, 1, 1, 2), (4, 32, 32, 1, 31, 1), (4, 32, 32, 4, 8, 1),
                                   (4, 32, 32, 3, 11, 1), (4, 32, 32, 7, 9, 1), (4, 32, 32, 8, 8, 1),
                                   (4, 32, 32, 5, 13, 1), (4, 32, 32, 4, 8, 3), (4, 16, 128, 1, 127, 1),
                                   (4, 32, 32, 8, 16, 1), (4, 32, 96, 1, 65, 2), (4, 32, 32, 8, 10, 2)])
def test_last_columns_kernel(shape):
    """Gram sizes 1, 2, 31..33, 63..65, 96, 127, 128, 130 and 160: below, at and above the 32
    columns of each slot of the last-columns kernel, and one or more column launches before it."""
    say(f"eigen-decomposition {shape} (s = {shape[3] * shape[4] * shape[5]})")
    check(shape)
    check(shape, rank_deficient=True)
