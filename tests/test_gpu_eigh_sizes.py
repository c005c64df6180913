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


@pytest.mark.parametrize("shape", [(4, 64, 64, 3, 43, 1), (4, 32, 32, 16, 16, 1), (4, 64, 64, 2, 43, 3),
                                   (8, 32, 32, 8, 8, 8), (4, 64, 64, 9, 19, 3), (4, 64, 64, 16, 16, 3),
                                   (6, 64, 64, 14, 11, 5), (5, 64, 64, 16, 16, 4), (4, 64, 64, 18, 19, 3),
                                   (6, 64, 64, 16, 16, 5), (4, 64, 64, 7, 61, 3)])
def test_resident_columns(shape):
    """Gram sizes 129, 256, 258, 512, 513, 768, 770, 1024, 1026 and 1280 of the resident
    reduction (the first size it takes, the last of and the first beyond every column slot,
    its largest), and 1281, which column launches take."""
    say(f"resident reduction {shape} (s = {shape[3] * shape[4] * shape[5]})")
    check(shape)


def test_resident_columns_rank_deficient():
    say("resident reduction, rank-deficient (s = 405)")
    check((6, 64, 64, 9, 9, 5), rank_deficient=True)


def problem(seed, n_irls=2):
    import workload
    return workload.make_problem(seed=seed, P=64, Q=64, T=8, K=2, R=4, N1=7, N2=7, M=4, n_irls=n_irls, n_cg=4)


def plan_of(pb):
    T, P, Q = pb.b.shape
    pl = slrx.Plan(P, Q, T, pb.N1, pb.N2, pb.M, slrx.make_params(lam=pb.lam, n_irls=pb.n_irls, n_cg=pb.n_cg))
    pl.set_kspace(pb.b)
    pl.set_mask(pb.S)
    return pl


def test_a_stalled_launch_is_repeated_by_column_launches():
    """A resident launch that gives up (forced from the host: its kernel leaves at once)
    costs time, not the result: alone, in a weights step and in a batch."""
    pbs = [problem(40 + i) for i in range(3)]
    plans = [plan_of(pb) for pb in pbs]
    refs = []
    for pl in plans:
        pl.run()
        pl.sync()
        refs.append(pl.images())
    say("forced stall, one plan")
    slrx.lib().slrx_fault_stall(1)
    plans[0].run()
    plans[0].sync()
    again = plans[0].images()
    # column launches round differently: FP64 reductions, then two steps of complex64 CG
    assert np.linalg.norm(again - refs[0]) <= 1e-5 * np.linalg.norm(refs[0])
    plans[0].run()
    plans[0].sync()
    np.testing.assert_array_equal(plans[0].images(), refs[0])
    say("forced stall, weights step")
    lam0, H0, E0 = plans[1].step_weights(100.0)
    slrx.lib().slrx_fault_stall(1)
    lam1, H1, E1 = plans[1].step_weights(100.0)
    s = lam0.size
    assert np.abs(lam1 - lam0).max() <= 80 * s * U * lam0[-1]
    assert np.linalg.norm(E1 - E0) <= 1e-6 * np.linalg.norm(E0)
    say("forced stall, batch")
    slrx.lib().slrx_fault_stall(1)
    slrx.run_batch(plans)
    for pl, ref in zip(plans, refs):
        img = pl.images()
        assert np.linalg.norm(img - ref) <= 1e-5 * np.linalg.norm(ref)
    say("forced stall, inputs replaced before the result was collected")
    slrx.lib().slrx_fault_stall(1)
    plans[2].run()
    import torch
    torch.cuda.synchronize()
    plans[2].set_mask(pbs[2].S)
    with pytest.raises(slrx.SlrxError) as ei:
        plans[2].sync()
    assert ei.value.name == "SLRX_EDEVICE"
    plans[2].run()
    plans[2].sync()
    np.testing.assert_array_equal(plans[2].images(), refs[2])
    for pl in plans:
        pl.close()


def test_concurrent_resident_launches_match_single_runs():
    """Plans run from several host threads at once, each on its own stream: resident
    launches share the chip without waiting for each other's workgroups, and every result
    is the one of the plan run alone, bit for bit."""
    import threading
    say("eight threads, s = 196")
    plans = [plan_of(problem(60 + i, n_irls=4)) for i in range(8)]
    refs = []
    for pl in plans:
        pl.run()
        pl.sync()
        refs.append(pl.images())
    errors = []

    def go(pl):
        try:
            for _ in range(3):
                pl.run()
                pl.sync()
        except Exception as e:  # pragma: no cover
            errors.append(e)

    threads = [threading.Thread(target=go, args=(pl,)) for pl in plans]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not errors
    for pl, ref in zip(plans, refs):
        np.testing.assert_array_equal(pl.images(), ref)
        pl.close()
