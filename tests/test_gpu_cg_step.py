"""CG iterations whose row pass finishes one iteration and begins the next (x, r and p in one
pass, alpha and beta from the finishing pass's dot products) against the complex128 oracle:
rows shorter than a block, the longest rows and the most frames, few iterations and many more
than convergence takes (where the residual is rounding noise and <r, r> predicted from the dot
products may be zero or negative), and residuals that are zero from the start.

Tolerance: one positive mask E in [0.2, 1] per pixel and lam = 1, so A = S + F E F^-1 has its
eigenvalues in [0.2, 2] and condition at most 10; a complex64 CG stops improving at a relative
error of about cond * eps32 * (a few), 10 * 6e-8 * 10 = 6e-6, taken as 1e-5 for the volume and
twice that for each frame."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import crandn, nrmse, say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")


def run(T, P, Q, S, b, E, n_cg):
    with slrx.Plan(P, Q, T, 3, 3, 1, slrx.make_params(lam=1.0, n_irls=1, n_cg=1)) as pl:
        pl.set_kspace(b)
        pl.set_mask(S)
        pl.step_cg(E[None].astype(np.complex64), n_cg)
        return pl.images()


@pytest.mark.parametrize("n_cg", (1, 2, 40))
@pytest.mark.parametrize("shape", ((1, 8, 8), (32, 8, 256), (3, 96, 16), (5, 256, 64), (2, 32, 160)))
def test_cg_step_matches_oracle(shape, n_cg):
    T, P, Q = shape
    say(f"cg step {shape} n_cg {n_cg}")
    rng = np.random.default_rng(7 * T + P + Q)
    S = (rng.random((T, P, Q)) < 0.5).astype(np.uint8)
    b = (S * crandn(rng, T, P, Q)).astype(np.complex64)
    E = 0.2 + 0.8 * rng.random((P, Q)).astype(np.float32)
    img = run(T, P, Q, S, b, E, n_cg)
    Sd = S.astype(np.float64)
    A = lambda v: Sd * v + oracle.dft2(E.astype(np.float64) * oracle.idft2(v))
    xk = oracle.cg(A, Sd * b, Sd * b.astype(np.complex128), n_cg)
    ref = oracle.idft2(xk)
    assert nrmse(img, ref) < 1e-5
    assert max(nrmse(img[t], ref[t]) for t in range(T)) < 2e-5


def test_cg_step_from_a_zero_residual():
    # b = 0, and a full mask without a penalty: the first residual is exactly zero, no step is taken
    T, P, Q = 2, 16, 32
    say("cg step, zero residual")
    rng = np.random.default_rng(5)
    S = np.ones((T, P, Q), np.uint8)
    b = crandn(rng, T, P, Q).astype(np.complex64)
    zero = np.zeros_like(b)
    E = np.full((P, Q), 0.5, np.float32)
    assert np.array_equal(run(T, P, Q, S, zero, E, 3), zero)
    one = run(T, P, Q, S, b, np.zeros((P, Q), np.float32), 0)
    assert np.array_equal(run(T, P, Q, S, b, np.zeros((P, Q), np.float32), 3), one)
