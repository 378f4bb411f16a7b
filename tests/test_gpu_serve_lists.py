"""Queries whose lists are built on the device and stay there: the same answers
as host-built ones, alone and mixed with them in a batch, where the lists kept
exceed their share of the budget, and beside queries that cannot be built."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402


@pytest.fixture(scope="module")
def tiny():
    S, Q, g = synth.configs.tiny()
    return S, Q, april.april_lists_to_device(april.april_build_lists(g, S.xy, S.voff, april.STRICT))


def answers(srv, queries):
    tickets = [srv.submit(q) for q in queries]
    out = []
    for t in tickets:
        try:
            r = srv.wait(t, 100)
            out.append((r.s_ids.copy(), r.verdict.copy()))
        except april.AprilError as e:
            out.append(e.code)
        srv.release(t)
    return out


def same(a, b):
    return a == b if isinstance(a, int) or isinstance(b, int) else all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("cells, budget", [(1, 1 << 28), (200, 1 << 28), (1, 1 << 20), (200, 1 << 20)])
def test_device_lists(tiny, cells, budget):
    S, Q, dS = tiny
    queries = [Q.polygon(k) for k in range(300)]
    bad = np.array([[50.0, 50.0], [50.5, 50.0], [50.0, 50.5]])   # outside the grid
    for k in (0, 7, 299):
        queries[k] = bad
    print(f"[serve lists] {cells} {budget}", flush=True)
    want = None
    for at in (0xFFFFFFFF, cells):
        srv = april.Server(dS, S.mbrs(), slots=2, mem_budget=budget, gpu_build_cells=at)
        try:
            # all at once twice (the first pass's lists are given back), then one by one
            passes = [answers(srv, queries), answers(srv, queries), [answers(srv, [q])[0] for q in queries[:40]]]
        finally:
            srv.close()
        if want is None:
            want = passes[0]
            assert want[0] == april.E_GRID and sum(not isinstance(w, int) for w in want) > 250
        for got in passes:
            for k, a in enumerate(got):
                assert same(a, want[k]), k
