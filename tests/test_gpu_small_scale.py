"""The eigen-decomposition and the reconstruction at small scales of the data: nothing in the
method has a unit, so a matrix or a k-space that is smaller by a power of two gives the scaled
result.  The Gram matrix is quadratic in the data, so its norm is easily below the rounding of
1, where a deflation tolerance that is not relative to the matrix drops its couplings.

Tolerances: eigenpairs as in the divide-and-conquer tests, c(s) = 120 s sqrt(s) u relative to
max |entry|, u = 2^-53.  A reconstruction whose lambda is scaled so that every quantity of the
CG is scaled by a power of two differs by FP64 rounding of the weights alone (the eigenvalues
and eps scale by 4^k, lambda by what makes lambda E invariant); the weights are then rounded to
complex64, and two outer iterations of CG keep the difference within 1e-5."""
import numpy as np
import pytest
import scipy.linalg

import workload
from tests.gpu_util import nrmse, say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")

SHAPES = {9: (3, 3, 1), 17: (17, 1, 1), 63: (9, 7, 1), 64: (8, 8, 1), 65: (13, 5, 1), 75: (5, 5, 3), 180: (6, 6, 5)}


@pytest.mark.parametrize("scale", [1e-6, 1e-12, 1e-15, 1e-30, 1e-76, 1e-140])
def test_tridiagonals_of_small_norm(scale):
    for s, (N1, N2, M) in SHAPES.items():
        say(f"divide and conquer, s = {s}, entries of size {scale}")
        rng = np.random.default_rng(s)
        d, e = rng.standard_normal(s), rng.standard_normal(s - 1)
        with slrx.Plan(32, 32, 5, N1, N2, M, slrx.make_params(n_irls=1, n_cg=1)) as pl:
            lam, Z = pl.step_tdeig(scale * d, scale * e)
        lam, Z = lam / scale, np.asarray(Z).real
        T = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
        tol = 120 * s * np.sqrt(s) * 2.0 ** -53 * max(np.abs(d).max(), np.abs(e).max())
        assert np.all(np.diff(lam) >= 0)
        assert np.abs(lam - scipy.linalg.eigvalsh(T)).max() <= tol
        assert np.linalg.norm(T @ Z - Z * lam) <= tol
        assert np.linalg.norm(Z.T @ Z - np.eye(s)) <= tol


@pytest.mark.parametrize("filt", [(5, 5, 3), (7, 7, 4)])
def test_reconstruction_scales_with_its_data(filt):
    """k-space times 2^-30: images times 2^-30, eps and lambda_max times 2^-60.  lambda E is
    invariant when lambda is scaled by 2^(60 (p/2 - 1)): E is a sum of (eigenvalue + eps)^(p/2-1)."""
    pb = workload.make_problem(seed=77, P=64, Q=64, T=8, K=2, R=4, N1=filt[0], N2=filt[1], M=filt[2], n_irls=2, n_cg=4)
    say(f"k-space times 2^-30, filter {filt}")
    out = []
    for k in (0, 30):
        prm = slrx.make_params(lam=pb.lam * 2.0 ** (2 * k * (0.6 / 2 - 1)), n_irls=2, n_cg=4)
        with slrx.Plan(64, 64, 8, *filt, prm) as pl:
            pl.set_kspace((pb.b * np.float32(2.0 ** -k)).astype(np.complex64))
            pl.set_mask(pb.S)
            pl.run()
            pl.sync()
            st = pl.stats()
            out.append((pl.images() * np.float32(2.0 ** k), np.array(st["eps"]) * 4.0 ** k,
                        np.array(st["lambda_max"]) * 4.0 ** k))
    (img0, eps0, lam0), (img1, eps1, lam1) = out
    e = nrmse(img1, img0)
    print(f"  NRMSE {e:.3e}", flush=True)
    np.testing.assert_allclose(lam1, lam0, rtol=1e-6)
    np.testing.assert_allclose(eps1, eps0, rtol=1e-6)
    assert e <= 1e-5
