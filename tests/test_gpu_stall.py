"""Resident tridiagonalisations that have to give up (slrx_fault_stall: a workgroup is missing
and every other one leaves after its bounded wait): what that may cost, and whom.  Results of
repeated runs are those of column launches, which round differently: FP64 reductions, then a
few steps of complex64 CG, 1e-5 as in the tests of the sizes."""
import time

import numpy as np
import pytest

import workload
from tests.gpu_util import nrmse, say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")


@pytest.fixture(autouse=True)
def disarm():
    yield
    slrx.lib().slrx_fault_stall(0)
    slrx.lib().slrx_fault_stall_wait(0)


def stall(n, ms=0):
    slrx.lib().slrx_fault_stall_wait(ms)
    slrx.lib().slrx_fault_stall(n)


def problem(seed, n_irls=6, N=7, M=4):
    return workload.make_problem(seed=seed, P=64, Q=64, T=8, K=2, R=4, N1=N, N2=N, M=M, n_irls=n_irls, n_cg=4)


def plan_of(pb, stream=None):
    T, P, Q = pb.b.shape
    pl = slrx.Plan(P, Q, T, pb.N1, pb.N2, pb.M, slrx.make_params(lam=pb.lam, n_irls=pb.n_irls, n_cg=pb.n_cg), stream=stream)
    pl.set_kspace(pb.b)
    pl.set_mask(pb.S)
    return pl


def run(pl):
    pl.run()
    pl.sync()
    return pl.images()


def test_a_run_waits_once():
    """Six decompositions that would each wait 200 ms: the run waits for the first one alone."""
    say("six stalled launches of 200 ms, one plan")
    pl = plan_of(problem(800))
    ref = run(pl)
    stall(6, 200)
    t0 = time.perf_counter()
    img = run(pl)
    dt = time.perf_counter() - t0
    say(f"{dt * 1e3:.0f} ms")
    assert 0.2 <= dt <= 0.6
    assert nrmse(img, ref) <= 1e-5
    stall(0)
    np.testing.assert_array_equal(run(pl), ref)  # the next run takes resident launches again
    pl.close()


def spectrum(pl):
    """The largest eigenvalue of every iteration, in FP64: images are rounded too coarsely to tell
    column launches from resident ones."""
    pl.run()
    pl.sync()
    return pl.stats()["lambda_max"]


def test_requests_wait_once():
    """The same for a server's group of two, whose runs give up together: that counts once, so a
    request after them takes resident launches (its own bits)."""
    say("two stalled launches of 300 ms, two requests")
    plans = [plan_of(problem(802 + i)) for i in range(3)]
    refs = [(spectrum(pl), pl.images()) for pl in plans]
    srv = slrx.Server(1 << 30, max_slots=4)
    try:
        stall(2, 300)  # the first two steps, whichever requests are in them
        t0 = time.perf_counter()
        for t in [srv.submit(pl) for pl in plans[:2]]:
            srv.wait(t)
        dt = time.perf_counter() - t0
        say(f"{dt * 1e3:.0f} ms")
        assert 0.3 <= dt <= 0.5
        stall(0)
        srv.wait(srv.submit(plans[2]))
    finally:
        srv.close()
    for pl, (lam, img) in zip(plans[:2], refs):
        assert pl.stats()["lambda_max"] != lam and nrmse(pl.images(), img) <= 1e-5
    assert plans[2].stats()["lambda_max"] == refs[2][0]
    np.testing.assert_array_equal(plans[2].images(), refs[2][1])
    for pl in plans:
        pl.close()


def test_a_stream_whose_launches_gave_up_twice_takes_column_launches():
    """Two give-ups on one stream: its next run takes column launches by itself (the bits of the
    repeated runs, no wait); other streams and a new plan's stream are not touched."""
    say("two stalled runs on one stream")
    pb = problem(810)
    pl, other = plan_of(pb), plan_of(pb)
    ref = spectrum(pl)
    stall(1)
    cols = spectrum(pl)
    np.testing.assert_allclose(cols, ref, rtol=1e-5)
    assert cols != ref
    assert spectrum(pl) == ref  # once is not enough
    stall(1)
    assert spectrum(pl) == cols
    stall(0)
    assert spectrum(pl) == cols
    lam0 = pl.step_weights(100.0)[0]
    assert spectrum(other) == ref
    lam1 = other.step_weights(100.0)[0]
    assert np.abs(lam0 - lam1).max() <= 80 * lam0.size * 2.0 ** -53 * lam0[-1] and not np.array_equal(lam0, lam1)
    pl.close()
    other.close()
    with plan_of(pb) as pl:  # most likely on the handle of a stream just destroyed
        assert spectrum(pl) == ref


def test_a_plan_made_for_every_run_on_a_callers_stream():
    """The stream is remembered, not the plan."""
    import torch
    say("two stalled plans on a caller's stream")
    pb = problem(810)
    st = torch.cuda.Stream()
    with plan_of(pb) as pl:
        ref = spectrum(pl)
    for _ in range(2):
        stall(1)
        with plan_of(pb, stream=st.cuda_stream) as pl:
            cols = spectrum(pl)
    stall(0)
    assert cols != ref
    with plan_of(pb, stream=st.cuda_stream) as pl:
        assert spectrum(pl) == cols


def test_a_server_whose_launches_gave_up_twice_takes_column_launches():
    say("two stalled requests of one server")
    pb = problem(810)
    with plan_of(pb) as pl:
        ref = spectrum(pl)
        srv = slrx.Server(1 << 30, max_slots=2)
        try:
            out = []
            for n in (0, 1, 1, 0):
                stall(n)
                srv.wait(srv.submit(pl))
                out.append(pl.stats()["lambda_max"])
        finally:
            srv.close()
    assert out[0] == ref and out[1] != ref
    assert out[2] == out[1] and out[3] == out[1]


def test_a_stream_kept_to_some_of_the_cus_takes_column_launches():
    """A resident launch waits for workgroups that a CU mask may never let run together."""
    import ctypes
    import torch
    say("a plan on a stream of half of the CUs")
    pb = problem(810)
    with plan_of(pb) as pl:
        ref = spectrum(pl)
        stall(1)
        cols = spectrum(pl)
        stall(0)
    hip = ctypes.CDLL([ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64" in ln][0])
    words = (torch.cuda.get_device_properties(0).multi_processor_count + 31) // 32
    mask = (ctypes.c_uint32 * words)(*([0xffffffff] * (words // 2)))
    h = ctypes.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(h), words, mask) == 0
    try:
        with plan_of(pb, stream=h.value) as pl:
            assert spectrum(pl) == cols and cols != ref
    finally:
        assert hip.hipStreamDestroy(h) == 0


def test_a_stalled_request_is_repeated_among_the_others():
    """The repeat of a served run does not hold the scheduler: a request that is two steps behind
    it finishes first, and one that joins its group meanwhile keeps its own bits."""
    say("a stalled request of 60 iterations, others beside it")
    pa, pb, pc = problem(810, n_irls=60), problem(813, n_irls=62, N=5, M=3), problem(814, n_irls=20)
    with plan_of(pa) as a, plan_of(pb) as b, plan_of(pc) as c:
        ref_c = spectrum(c)
        ref_a = spectrum(a)
        stall(1)
        cols = spectrum(a)
        assert cols != ref_a
        srv = slrx.Server(1 << 30, max_slots=4)
        try:
            stall(1)
            ta, tb = srv.submit(a), srv.submit(b)
            srv.wait(tb)
            tc = srv.submit(c)
            for t in (ta, tc):
                srv.wait(t)
            ia, ib, ic = (srv.info(t) for t in (ta, tb, tc))
        finally:
            srv.close()
        assert ib["t_done"] < ia["t_done"]
        assert ic["t_admit"] < ia["t_done"]
        assert a.stats()["lambda_max"] == cols and c.stats()["lambda_max"] == ref_c
        assert spectrum(a) == ref_a  # alone again, on its own stream
