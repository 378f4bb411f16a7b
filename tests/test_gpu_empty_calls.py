"""Calls of no pairs: counts are zeros and there is no error, whatever the
lists are (calls on long lists are screened however few pairs they have)."""

import numpy as np
import pytest

from synth.grid import Grid
from synth.intervals import ListSet, random_lists, sub_lists

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402

GRID, COARSER = Grid(0.0, 0.0, 1.0, 10), Grid(0.0, 0.0, 1.0, 9)


def lists(grid, n):
    rng = np.random.default_rng(n)
    A = [random_lists(rng, n, 0, 16 * n) for _ in range(3)]
    a, f = ListSet.from_lists(A), ListSet.from_lists([sub_lists(rng, *x, p=0.5) for x in A])
    return april.april_lists_from_arrays(grid, a.off, a.start, a.end, f.off, f.start, f.end)


@pytest.mark.parametrize("n", [20, 600, 5000])
def test_no_pairs(n):
    print(f"[empty] {n}", flush=True)
    host = lists(GRID, n)
    L, M = april.april_lists_to_device(host), april.april_lists_to_device(lists(COARSER, n))
    V = april.april_lists_to_device(host, april.CODEC_VBYTE)
    xy = np.array([[0.25, 0.25], [0.5, 0.5], [0.75, 0.25]])
    C = april.april_cells_to_device(april.april_build_cells(GRID, xy, np.array([0, 3], np.uint64)))
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    calls = [lambda v, c: april.april_filter_within(L, L, none, none, v, c),
             lambda v, c: april.april_filter_linestrings(L, C, none, none, v, c),
             lambda v, c: april.april_filter_mixed(L, M, none, none, v, c),
             lambda v, c: april.april_filter_mixed(L, L, none, none, v, c),
             lambda v, c: april.april_filter_pairs(L, L, none, none, v, c),
             lambda v, c: april.april_filter_pairs(L, L, none, none, v, c, schedule=april.SCHED_BATCHED),
             lambda v, c: april.april_filter_pairs(V, V, none, none, v, c, schedule=april.SCHED_BATCHED)]
    for k, call in enumerate(calls):
        c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
        call(torch.empty(0, dtype=torch.uint8, device="cuda"), c)
        torch.cuda.synchronize()
        assert c.tolist() == [0, 0, 0], k
        call(torch.empty(0, dtype=torch.uint8, device="cuda"), None)
        torch.cuda.synchronize()
