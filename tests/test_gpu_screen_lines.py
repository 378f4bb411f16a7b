"""Polygon-linestring calls at the edges of screening's parts and lists of open
pairs, and on lists whose F-intervals lie outside A."""

import numpy as np
import pytest

import oracle
from synth.grid import Grid
from synth.intervals import ListSet, random_lists, sub_lists

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


@pytest.mark.parametrize("sizes", [[62, 63, 64, 255, 256, 257], [1, 40, 700, 2047, 2049, 5000]])
def test_in_parts(sizes):
    """More pairs than are screened at a time: the same ones over and over."""
    print(f"[lines] parts {sizes}", flush=True)
    rng = np.random.default_rng(50 + len(sizes) + sizes[0])
    A = [random_lists(rng, sizes[k % len(sizes)], 0, IDS if k % 2 else max(16 * sizes[k % len(sizes)], IDS >> 4))
         for k in range(24)]
    P, LP = polygons(A, [sub_lists(rng, *a, p=0.3) for a in A])
    C, LC = walks(rng, 24)
    p, l = (rng.integers(0, 24, 9001).astype(np.uint32) for _ in range(2))
    p.sort()
    want = oracle.filter_linestrings(LP, LC, p, l)
    assert set(np.unique(want)) == {0, 1, 2}
    times = (1 << 24) // len(p) + 7
    v, counts = call(P, C, dev(p).repeat(times), dev(l).repeat(times))
    assert bool((v.view(times, -1) == torch.from_numpy(want).cuda()).all())
    assert counts == (np.bincount(want, minlength=3) * times).tolist()


@pytest.mark.parametrize("sizes, n", [([3, 40], 70_000), ([3], 1_100_000), ([600], 300_000), ([600], 600_000),
                                      ([3, 600], 1_200_000)])
def test_open_lists(sizes, n):
    """Every pair is left open (no F-intervals, a cell that all meet): lists that
    hold them all, and lists of either kind that overflow."""
    print(f"[lines] open {sizes} {n}", flush=True)
    rng = np.random.default_rng(n)
    C, LC = walks(rng, 8)
    cell = np.uint32(LC.ids[0])
    none = (np.zeros(0, np.uint32), np.zeros(0, np.uint32))
    A = []
    for k in range(40):
        m = sizes[k % len(sizes)]
        s = np.unique(np.append(rng.choice(IDS // 8, m, replace=False).astype(np.uint32) * 8 + 1, cell))
        A.append((s, s + np.uint32(1)))
    P, _ = polygons(A, [none] * 40)
    p = rng.integers(0, 40, n).astype(np.uint32)
    v, counts = call(P, C, dev(p), dev(np.zeros(n, np.uint32)))
    assert int((v != april.INDECISIVE).sum()) == 0
    assert counts == [0, 0, n]
