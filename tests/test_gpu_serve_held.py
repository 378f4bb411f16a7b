"""Device memory of queries whose lists were built on the device: given back
when a query fails for its size, though its ticket is not released, and when
queries are cancelled at any stage."""

import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402

SPACE = (-0.125, -0.125, 1.25)


def spikes(n, out=0.4):
    """A star of n long spikes: some 20,000 cells along every edge."""
    t = 2 * np.pi * np.arange(2 * n) / (2 * n)
    r = np.where(np.arange(2 * n) % 2, 0.05, out)
    xy = np.stack([0.5 + r * np.cos(t), 0.5 + r * np.sin(t)], 1)
    return np.round(xy * 2.0 ** 30) * 2.0 ** -30


def settled():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.fixture(scope="module")
def collection():
    S, _, _ = synth.configs.tiny()
    g = SPACE + (16,)
    return S, april.april_lists_to_device(april.april_build_lists(g, S.xy, S.voff, april.STRICT))


def returns(free, slack=3 << 20):
    """Does the device's free memory come back to `free` (less some pages)?"""
    for _ in range(100):
        if settled() >= free - slack:
            return True
        time.sleep(0.05)
    return False


def test_failed_query_holds_nothing(collection):
    S, dS = collection
    q = spikes(60)
    info = april.april_build_lists(SPACE + (16,), q, np.array([0, len(q)], np.uint64)).info()
    size = info.n_a + info.n_f
    # a slot takes 0.75 of the query's intervals, the kept lists' share 1.25 of its bytes
    srv = april.Server(dS, S.mbrs(), slots=2, mem_budget=40 * size, gpu_build_cells=1)
    try:
        assert srv.stats()["cap_intervals"] < size and 8 * size > 8 << 20

        def fail():
            t = srv.submit(q)
            with pytest.raises(april.AprilError) as e:
                srv.wait(t, 60)
            assert e.value.code == april.E_NOMEM
            return t

        srv.release(fail())
        free = settled()
        kept = [fail() for _ in range(3)]   # not released
        assert returns(free)
        # and other queries are served beside them
        t = srv.submit(S.polygon(0))
        assert 0 in srv.wait(t, 60).s_ids
        for t in kept:
            srv.release(t)
    finally:
        srv.close()


def test_cancelled_queries_hold_nothing(collection):
    S, dS = collection
    q = spikes(12)
    srv = april.Server(dS, S.mbrs(), slots=2, gpu_build_cells=1)
    try:
        t = srv.submit(q)
        srv.wait(t, 60)
        srv.release(t)
        free = settled()
        for wait in (0.0, 0.001, 0.003, 0.01):
            tickets = [srv.submit(q) for _ in range(12)]
            time.sleep(wait)
            for t in tickets:
                srv.cancel(t)
        assert returns(free)
        t = srv.submit(S.polygon(0))
        assert 0 in srv.wait(t, 60).s_ids
        srv.release(t)
    finally:
        srv.close()
