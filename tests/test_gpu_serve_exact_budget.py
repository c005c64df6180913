"""A request whose device bytes are exactly the server's budget is admitted once the server is
idle, whatever ran before: idle plans are evicted and the engine's shared buffers, the tables
of the grouped launches among them, are given back."""
import numpy as np
import pytest

import workload
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")


@pytest.mark.parametrize("grouping", [0, 1])
def test_exact_fit_after_grouped_requests(grouping):
    big = workload.make_problem(seed=81, P=64, Q=64, T=8, K=2, R=4, N1=7, N2=7, M=4, n_irls=2, n_cg=4)
    small = [workload.make_problem(seed=82 + i, P=32, Q=32, T=6, K=1, R=4, N1=5, N2=5, M=3, n_irls=60, n_cg=4)
             for i in range(2)]

    def submit(srv, pb):
        return srv.submit_data(pb.b, pb.S, pb.N1, pb.N2, pb.M,
                               slrx.make_params(lam=pb.lam, n_irls=pb.n_irls, n_cg=pb.n_cg))

    say(f"exact budget, CG {'grouped' if grouping else 'per problem'}")
    slrx.set_cg_grouping(grouping)
    try:
        srv = slrx.Server(1 << 30)
        t = submit(srv, big)
        srv.wait(t)
        need, ref = srv.info(t)["bytes"], srv.fetch(t, big.b.shape)
        srv.close()
        srv = slrx.Server(need, max_slots=2)
        try:
            ts = [submit(srv, pb) for pb in small]
            for t in ts:
                srv.wait(t)
            a, b = (srv.info(t) for t in ts)
            assert a["t_admit"] < b["t_done"] and b["t_admit"] < a["t_done"]  # they shared launches
            t = submit(srv, big)
            assert srv.wait_for(t, 20.0)
            np.testing.assert_array_equal(srv.fetch(t, big.b.shape), ref)
        finally:
            srv.close()
    finally:
        slrx.set_cg_grouping(-1)
