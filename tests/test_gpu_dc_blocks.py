"""The divide and conquer below 64 entries on tridiagonals that reach its special cases: blocks
that split, equal and clustered eigenvalues, couplings and diagonals near both ends of the
exponent range (where the rotations leave the fast square root), and sizes on both sides of
every base block (8 entries), half and full subtree (64).

Tolerance: every merge and rotation is backward stable, so eigenvalues are within c(s) u ||T||
of LAPACK's and ||T Z - Z lambda||, ||Z^T Z - I|| within c(s) u (times ||T||), with
c(s) = 40 s for both sides and another sqrt(s) for the Frobenius norms, u = 2^-53."""
import numpy as np
import pytest
import scipy.linalg

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")

SHAPES = {1: (1, 1, 1), 2: (2, 1, 1), 7: (7, 1, 1), 8: (4, 2, 1), 9: (3, 3, 1), 16: (4, 4, 1), 17: (17, 1, 1),
          33: (11, 3, 1), 63: (9, 7, 1), 64: (8, 8, 1), 65: (13, 5, 1)}


def matrix(kind, s, rng):
    d, e = rng.standard_normal(s), rng.standard_normal(max(s - 1, 0))
    if kind == "split":
        e[::3] = 0.0
    elif kind == "equal":
        d[:], e[:] = 2.0, 0.0
    elif kind == "clustered":
        d = np.ones(s) + 1e-15 * d
        e *= 1e-9
    elif kind == "graded":
        g = 10.0 ** -np.linspace(0, 14, s)
        d, e = d * g, e * np.sqrt(g[:-1] * g[1:]) if s > 1 else e
    elif kind == "wilkinson":
        d, e = np.abs(np.arange(s) - (s - 1) / 2.0), np.ones(max(s - 1, 0))
    elif kind == "tiny":
        d, e = 1e-140 * d, 1e-140 * e
    elif kind == "huge":
        d, e = 1e140 * d, 1e140 * e
    return d, e


@pytest.mark.parametrize("kind", ("random", "split", "equal", "clustered", "graded", "wilkinson", "tiny", "huge"))
def test_small_blocks(kind):
    for s, (N1, N2, M) in SHAPES.items():
        if kind == "tiny" and s > 8:
            continue  # merges deflate couplings below rounding of 1: the base blocks alone
        say(f"divide and conquer, {kind}, s = {s}")
        d, e = matrix(kind, s, np.random.default_rng(s))
        with slrx.Plan(32, 32, 4, N1, N2, M, slrx.make_params(n_irls=1, n_cg=1)) as pl:
            lam, Z = pl.step_tdeig(d, e)
        norm = max(np.abs(d).max(), np.abs(e).max() if s > 1 else 0.0) or 1.0
        T = np.diag(d / norm) + (np.diag(e / norm, 1) + np.diag(e / norm, -1) if s > 1 else 0.0)
        ref = scipy.linalg.eigvalsh(T)
        lam, Z = lam / norm, np.asarray(Z).real
        tol = 40 * s * np.sqrt(s) * 2.0 ** -53 * 3  # ||T|| <= 3 max |entry|
        assert np.all(np.diff(lam) >= 0)
        assert np.abs(lam - ref).max() <= tol
        assert np.linalg.norm(T @ Z - Z * lam) <= tol
        assert np.linalg.norm(Z.T @ Z - np.eye(s)) <= tol
