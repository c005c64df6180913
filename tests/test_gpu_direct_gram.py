"""The Gram matrix of IRLS-direct (k_dgram: 64 x 64 tiles, chunks of 16 lifted rows split
over workgroups) where its tiles, chunks and splits end: the largest eigenvalue of the first
outer iteration, in FP64, and the images, against the oracle.

Tolerance of the eigenvalue: the entries are sums of `rows` products of exact complex64
values in FP64, so ||dR|| <= rows u sum |x|^2 <= rows s u lambda_max (both sides, any order),
and the eigensolver adds at most 40 s u lambda_max (u = 2^-53).  Images: 1e-4 relative, the
bar of the direct method's parity tests."""
import numpy as np
import pytest

import oracle
import workload
from tests.gpu_util import nrmse, say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")


@pytest.mark.parametrize("P,Q,T,N1,N2,M", [
    (16, 16, 2, 16, 4, 2),     # 13 rows, fewer than one chunk; s = 128, two whole tiles
    (32, 16, 4, 8, 8, 1),      # s = 64, one whole tile; wrapped shifts on both axes
    (32, 32, 3, 5, 13, 1),     # s = 65, one column into the second tile
    (16, 32, 5, 3, 7, 3),      # s = 63, one short of a tile
    (32, 64, 6, 3, 3, 2),      # s = 18, many splits of one tile, the last one ragged
    (64, 32, 4, 6, 11, 2),     # s = 132, six tiles
])
def test_gram_at_tile_and_split_edges(P, Q, T, N1, N2, M):
    s, rows = N1 * N2 * M, (T - M + 1) * (P - N1 + 1) * (Q - N2 + 1)
    say(f"direct gram {P}x{Q}x{T} {N1}x{N2}x{M}: {rows} x {s}")
    pb = workload.make_problem(seed=300 + s, P=P, Q=Q, T=T, K=2, R=2, N1=N1, N2=N2, M=M, n_irls=2, n_cg=3, phase=True)
    prm = slrx.make_params(lam=pb.lam, n_irls=2, n_cg=3, direct=True)
    with slrx.Plan(P, Q, T, N1, N2, M, prm) as pl:
        pl.set_kspace(pb.b)
        pl.set_mask(pb.S)
        pl.run()
        pl.sync()
        img, st = pl.images(), pl.stats()
    lam = np.linalg.eigvalsh(oracle.gram_direct(pb.S * pb.b.astype(np.complex128), N1, N2, M))[-1]
    assert abs(st["lambda_max"][0] - lam) <= (rows * s + 40 * s) * 2.0 ** -53 * lam
    assert nrmse(img, oracle.irls_direct(pb.b, pb.S, N1, N2, M, pb.lam, 2, 3)) <= 1e-4
