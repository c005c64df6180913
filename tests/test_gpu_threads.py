"""Host threads that make, run and close plans of their own at once: a thread's first runs
capture the CG while the others copy synchronously (tables of a new plan, status of a finished
run), which HIP refuses beside a capture, to the loss of both.  Results are those of the plans
alone, bit for bit."""
import threading

import numpy as np
import pytest

import workload
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")


def run_new_plan(seed):
    pb = workload.make_problem(seed=seed, P=32, Q=32, T=6, K=1, R=4, N1=3, N2=3, M=2, n_irls=4, n_cg=3)
    with slrx.Plan(32, 32, 6, 3, 3, 2, slrx.make_params(lam=pb.lam, n_irls=4, n_cg=3)) as pl:
        pl.set_kspace(pb.b)
        pl.set_mask(pb.S)
        pl.run()
        pl.sync()
        pl.stats()
        return pl.images()


def test_new_plans_in_eight_threads():
    say("eight threads, twelve new plans each")
    seeds = [900 + i for i in range(8)]
    refs = [run_new_plan(s) for s in seeds]
    errors, bad = [], []
    start = threading.Barrier(8)

    def go(s, ref):
        try:
            start.wait(60)
            for _ in range(12):
                if not np.array_equal(run_new_plan(s), ref):
                    bad.append(s)
        except Exception as e:  # pragma: no cover
            errors.append(e)

    threads = [threading.Thread(target=go, args=a) for a in zip(seeds, refs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not errors, errors[:2]
    assert not bad
