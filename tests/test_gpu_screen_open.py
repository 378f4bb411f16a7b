"""Screened calls in which stretches of open pairs and of decided ones follow
each other, so that waves give screening up and take it up again, with lists of
open pairs that hold all of them and that do not."""

import numpy as np
import pytest

import oracle
from synth.grid import Grid
from synth.intervals import ListSet, random_lists, sub_lists

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402

G, IDS, N = Grid(0.0, 0.0, 1.0, 10), 1 << 20, 64
NONE = (np.zeros(0, np.uint32), np.zeros(0, np.uint32))


def objects(rng, sizes):
    """Objects 0 .. 31 meet in A only, 32 .. 63 in F too (and lie apart from some)."""
    A, F = [], []
    for k in range(N):
        m = sizes[k % len(sizes)]
        a = random_lists(rng, m, 0, 16 * m) if k % 8 else random_lists(rng, m, IDS // 2, IDS // 2 + 16 * m)
        A.append(a)
        F.append(NONE if k < 32 else sub_lists(rng, *a, p=0.9))
    a, f = ListSet.from_lists(A), ListSet.from_lists(F)
    return oracle.Lists(a.off, a.start, a.end, f.off, f.start, f.end)


def stretches(rng, n, m):
    """Pair ids with first ids below 32 for some thousands, then above, ...; the
    second ids below m."""
    r = np.empty(n, np.uint32)
    at, low = 0, True
    while at < n:
        k = min(n - at, int(rng.integers(100, 200_000)))
        r[at:at + k] = rng.integers(0, 32, k) + (0 if low else 32)
        at, low = at + k, not low
    return r, rng.integers(0, m, n).astype(np.uint32)


@pytest.mark.parametrize("kind", ["batched", "plain", "within", "lines"])
@pytest.mark.parametrize("sizes", [[1, 3, 8], [3, 40, 200], [20, 700]])   # (the shortest: not screened at 2.6M)
@pytest.mark.parametrize("n", [600_000, 2_600_000])
def test_stretches(kind, sizes, n):
    print(f"[stretches] {kind} {sizes} {n}", flush=True)
    rng = np.random.default_rng(n + len(sizes))
    L = objects(rng, sizes)
    h = april.april_lists_from_arrays(G, L.offA, L.sA, L.eA, L.offF, L.sF, L.eF)
    R, every = april.april_lists_to_device(h), np.arange(N, dtype=np.uint32)
    fn, kw = april.april_filter_pairs, {}
    if kind == "lines":
        lines = [np.round((rng.random(2) * 0.1 + 0.01 + np.cumsum(rng.random((k + 2, 2)) * 2.0 ** -8, axis=0)) * 2.0 ** 30)
                 * 2.0 ** -30 for k in range(24)]
        C = april.april_build_cells(G, np.concatenate(lines),
                                    np.concatenate([[0], np.cumsum([len(x) for x in lines])]).astype(np.uint64))
        S, m, fn = april.april_cells_to_device(C), 24, april.april_filter_linestrings
        p, q = np.repeat(every, m), np.tile(np.arange(m, dtype=np.uint32), N)
        table = oracle.filter_linestrings(L, oracle.Cells(*C.export()), p, q)
    else:
        S, m = R, N
        p, q = np.repeat(every, N), np.tile(every, N)
        table = (oracle.filter_within if kind == "within" else oracle.filter_pairs)(L, L, p, q)
        if kind == "within":
            fn = april.april_filter_within
        else:
            kw = {"schedule": april.SCHED_PLAIN if kind == "plain" else april.SCHED_BATCHED}
    table = torch.from_numpy(table).cuda().view(N, m)
    r, s = stretches(rng, n, m)
    rt, st = (torch.from_numpy(x.view(np.int32)).cuda() for x in (r, s))
    want = table[rt.long(), st.long()]
    v = torch.full((n,), 77, dtype=torch.uint8, device="cuda")
    c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    for _ in range(2):
        fn(R, S, rt, st, v, c, **kw)
    torch.cuda.synchronize()
    assert torch.equal(v, want)
    assert c.tolist() == torch.bincount(want.long(), minlength=3).tolist()
