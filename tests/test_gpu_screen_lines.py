"""Screened polygon-linestring calls: lists whose F-intervals lie outside A."""

import numpy as np
import pytest

import oracle
from synth.grid import Grid
from synth.intervals import ListSet, random_lists

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402

G, IDS = Grid(0.0, 0.0, 1.0, 10), 1 << 20


def walks(rng, n):
    """n linestrings of 1 to 4,000 short steps: (device cells, the oracle's)."""
    steps, lines = [1, 2, 20, 40, 60, 100, 300, 4000], []
    for k in range(n):
        walk = rng.random(2) + np.cumsum(rng.normal(0, 2.0 ** -9, (steps[k % len(steps)] + 1, 2)), axis=0)
        lines.append(np.round(np.clip(walk, 0.01, 0.99) * 2.0 ** 30) * 2.0 ** -30)
    voff = np.concatenate([[0], np.cumsum([len(x) for x in lines])]).astype(np.uint64)
    C = april.april_build_cells(G, np.concatenate(lines), voff, april.STRICT)
    return april.april_cells_to_device(C), oracle.Cells(*C.export())


def polygons(A, F, validate=True):
    a, f = ListSet.from_lists(A), ListSet.from_lists(F)
    h = april.april_lists_from_arrays(G, a.off, a.start, a.end, f.off, f.start, f.end, validate=validate)
    return april.april_lists_to_device(h), oracle.Lists(a.off, a.start, a.end, f.off, f.start, f.end)


def call(P, C, p, l):
    v = torch.full((len(p),), 77, dtype=torch.uint8, device="cuda")
    c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    april.april_filter_linestrings(P, C, p, l, v, c)
    torch.cuda.synchronize()
    return v, c.tolist()


def dev(x):
    return torch.from_numpy(x.view(np.int32)).cuda()


@pytest.mark.parametrize("sizes", [[5, 40, 200, 600], [5, 40, 200]])
def test_f_outside_a(sizes):
    """The cells count in F only where they meet A too, screened (one call) and
    not (calls of fewer pairs)."""
    print(f"[lines] outside {sizes}", flush=True)
    rng = np.random.default_rng(len(sizes))
    A = [random_lists(rng, sizes[k % len(sizes)], 0, IDS // 2) for k in range(40)]
    F = [random_lists(rng, sizes[k % len(sizes)], 0, IDS) for k in range(40)]
    P, _ = polygons(A, F, validate=False)
    C, _ = walks(rng, 40)
    p, l = (rng.integers(0, 40, 9000).astype(np.uint32) for _ in range(2))
    p.sort()
    parts = [call(P, C, dev(p[i:i + 4500]), dev(l[i:i + 4500])) for i in (0, 4500)]
    v, counts = call(P, C, dev(p), dev(l))
    assert torch.equal(v, torch.cat([x[0] for x in parts]))
    assert counts == [sum(x) for x in zip(*(x[1] for x in parts))]
