"""Grouped weight updates of batches (one launch per kernel for all problems of one filter)
against the same problems run alone, bit for bit: the blocks of a problem do what its own
launches do, so no tolerance applies.  Uneven frames and echo counts (the grids are the
largest over the problems), GIRAF beside the hybrid lifting, other filters, coils and
parameters in the same batch, filters beyond the spectral route, and problems that stop at
different outer iterations (each keeps its own)."""
import numpy as np
import pytest

import workload
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")


def plan(seed, P, Q, T, N1, N2, M, n_irls=3, giraf=False, p=0.6, gamma=1.4, coils=0):
    kw = dict(P=P, Q=Q, T=T, K=2, R=4, N1=N1, N2=N2, M=M, n_irls=n_irls, n_cg=3)
    pb = workload.make_mc_problem(seed=seed, ncoils=coils, **kw) if coils else workload.make_problem(seed=seed, **kw)
    pl = slrx.Plan(P, Q, T, N1, N2, M, slrx.make_params(lam=pb.lam, n_irls=n_irls, n_cg=3, giraf=giraf, p=p, gamma=gamma))
    pl.set_mask(pb.S)
    if coils:
        pl.set_coils(pb.coils, pb.b)
    else:
        pl.set_kspace(pb.b)
    return pl


BATCHES = {
    "uneven frames, one filter": [(64, 32, 6, 3, 5, 2), (8, 256, 4, 3, 5, 2), (96, 160, 9, 3, 5, 2), (16, 8, 2, 3, 5, 2)],
    "two filters of one Gram size": [(32, 32, 6, 3, 5, 2), (64, 32, 6, 5, 3, 2), (32, 64, 5, 3, 5, 2), (32, 32, 5, 5, 3, 2),
                                     (32, 32, 5, 6, 5, 1)],
    "beyond the spectral route": [(32, 32, 8, 3, 3, 6), (32, 64, 9, 3, 3, 6), (64, 32, 8, 2, 27, 1), (32, 32, 4, 2, 27, 1)],
}


@pytest.mark.parametrize("grouping", [0, 1])
@pytest.mark.parametrize("name", list(BATCHES))
def test_grouped_weights_match_single_runs(name, grouping):
    say(f"{name}, CG {'grouped' if grouping else 'per problem'}")
    plans = [plan(500 + i, *shape, n_irls=2 + i % 3) for i, shape in enumerate(BATCHES[name])]
    if name == "uneven frames, one filter":
        plans.append(plan(520, 32, 32, 6, 3, 5, 2, giraf=True))
        plans.append(plan(521, 32, 32, 6, 3, 5, 2, p=0.9, gamma=1.7))
        plans.append(plan(522, 32, 32, 6, 3, 5, 2, coils=3))
    refs, stats = [], []
    for pl in plans:
        pl.run()
        pl.sync()
        refs.append(pl.images())
        stats.append(pl.stats())
    slrx.set_cg_grouping(grouping)
    try:
        for _ in range(2):
            slrx.run_batch(plans)
            for i, pl in enumerate(plans):
                np.testing.assert_array_equal(pl.images(), refs[i], err_msg=f"problem {i}")
                st = pl.stats()
                for k in ("eps", "lambda_max", "cg_rr_final"):
                    assert st[k] == stats[i][k], (i, k)
    finally:
        slrx.set_cg_grouping(-1)
        for pl in plans:
            pl.close()


def test_more_problems_than_one_grouped_launch_takes():
    """66 problems: the grouped launches take at most 64 at a time."""
    say("66 problems")
    plans = [plan(600 + i, (8, 16, 32)[i % 3], 16, 3, 2, 2, 1, n_irls=2) for i in range(66)]
    refs = []
    for pl in plans:
        pl.run()
        pl.sync()
        refs.append(pl.images())
    for grouping in (0, 1):
        slrx.set_cg_grouping(grouping)
        try:
            slrx.run_batch(plans)
        finally:
            slrx.set_cg_grouping(-1)
        for pl, ref in zip(plans, refs):
            np.testing.assert_array_equal(pl.images(), ref)
    for pl in plans:
        pl.close()
