"""Resident tridiagonalisations of several streams at once: their workgroups wait for each
other, so launches that do not fit the chip together have to run one after another.  Results
are then those of the plans run alone, bit for bit (a launch that has to give up is repeated by
column launches, which round differently)."""
import threading

import numpy as np
import pytest

import workload
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

slrx = pytest.importorskip("paper_1704_04511_amd")


def plan(seed, N2=73, stream=None):
    """Gram size 2 N2: N2 workgroups of two rows each."""
    pb = workload.make_problem(seed=seed, P=32, Q=96, T=4, K=1, R=4, N1=1, N2=N2, M=2, n_irls=4, n_cg=3)
    pl = slrx.Plan(32, 96, 4, 1, N2, 2, slrx.make_params(lam=pb.lam, n_irls=4, n_cg=3), stream=stream)
    pl.set_kspace(pb.b)
    pl.set_mask(pb.S)
    return pl


def together(jobs):
    errors = []

    def go(job):
        try:
            job()
        except Exception as e:  # pragma: no cover
            errors.append(e)

    threads = [threading.Thread(target=go, args=(j,)) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not errors, errors


def test_launches_that_fill_one_xcd_more_than_the_others():
    """Seven launches of 73 workgroups: fewer than the 512 of the chip, but ten on the first XCD
    for each launch, of 64 that it holds."""
    say("seven streams, 73 workgroups each")
    plans = [plan(700 + i) for i in range(7)]
    refs = []
    for pl in plans:
        pl.run()
        pl.sync()
        refs.append(pl.images())

    def job(pl):
        for _ in range(4):
            pl.run()
            pl.sync()

    together([lambda pl=pl: job(pl) for pl in plans])
    for pl, ref in zip(plans, refs):
        np.testing.assert_array_equal(pl.images(), ref)
        pl.close()


def test_the_per_thread_stream_is_another_stream_in_every_thread():
    """Plans on hipStreamPerThread (handle 2): eight threads, 88 workgroups each, on eight
    streams behind one handle, so that they do not wait for each other by themselves."""
    say("eight threads on hipStreamPerThread, 88 workgroups each")
    refs = []
    for i in range(8):
        with plan(720 + i, N2=88) as pl:
            pl.run()
            pl.sync()
            refs.append(pl.images())
    out = [None] * 8

    def job(i):
        with plan(720 + i, N2=88, stream=2) as pl:
            for _ in range(4):
                pl.run()
                pl.sync()
            out[i] = pl.images()

    together([lambda i=i: job(i) for i in range(8)])
    for a, ref in zip(out, refs):
        np.testing.assert_array_equal(a, ref)


@pytest.mark.parametrize("N2", [73, 53])
def test_a_run_does_not_disturb_a_capture_elsewhere(N2):
    """Runs enqueued while the program captures a stream of its own, in the default capture mode:
    from another thread and from the capturing thread, on the plans' streams (Gram size 146, and
    106, whose column launches are still being tuned)."""
    import torch
    say(f"runs enqueued during a capture, s = {2 * N2}")
    pa, pb = plan(740, N2), plan(741, N2)
    refs = []
    for pl in (pa, pb):
        for _ in range(2):  # the second run replays the captured CG
            pl.run()
            pl.sync()
        refs.append(pl.images())
    x = torch.ones(1 << 16, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = x * 2
        together([pa.run])
        pb.run()
        y = y + 1
    for pl, ref in zip((pa, pb), refs):
        pl.sync()
        np.testing.assert_array_equal(pl.images(), ref)
        pl.close()
    g.replay()
    torch.cuda.synchronize()
    assert float(y[0]) == 3.0
