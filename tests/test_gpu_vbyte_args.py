"""Compressed filter calls: those that are refused write nothing; the decode
cache in calls that are screened."""

import numpy as np
import pytest

import oracle
from synth.intervals import ListSet, random_lists, sub_lists

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402

GRID = (0.0, 0.0, float(1 << 16) * 2.0 ** -30 * (1 << 16), 16)


@pytest.mark.parametrize("bad", ["cache", "no workspace", "tile", "chunk"])
@pytest.mark.parametrize("n", [40, 2000])
def test_refused(n, bad):
    print(f"[vbyte args] {n} {bad}", flush=True)
    rng = np.random.default_rng(n)
    A = [random_lists(rng, n, 0, 16 * n) for _ in range(4)]
    a, f = ListSet.from_lists(A), ListSet.from_lists([sub_lists(rng, *x, p=0.5) for x in A])
    V = april.april_lists_to_device(april.april_lists_from_arrays(GRID, a.off, a.start, a.end, f.off, f.start, f.end),
                                    april.CODEC_VBYTE)
    r = torch.randint(0, 4, (20_000,), dtype=torch.int32, device="cuda")
    v = torch.full((20_000,), 77, dtype=torch.uint8, device="cuda")
    c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    ws = torch.empty(april.april_filter_workspace_size(20_000, flags=april.WS_DECODE_CACHE) - 1, dtype=torch.uint8,
                     device="cuda")
    kw = {"cache": {"flags": april.WS_DECODE_CACHE, "workspace": ws}, "no workspace": {"flags": april.WS_DECODE_CACHE},
          "tile": {"tile": 300}, "chunk": {"chunk": 5}}[bad]
    with pytest.raises(april.AprilError) as e:
        april.april_filter_pairs(V, V, r, r, v, c, schedule=april.SCHED_BATCHED, **kw)
    assert e.value.code == april.E_INVALID
    torch.cuda.synchronize()
    assert bool((v == 77).all()) and c.tolist() == [-1, -1, -1]


@pytest.mark.parametrize("run", [4, 11, 12, 13, 100])
def test_cache_of_screened_calls(run):
    """Pairs that screening leaves open, in runs that share their R object, with
    the caller's decode cache (which takes runs of 12 in a grab): between objects
    whose lists interleave, some with one overlap."""
    print(f"[vbyte cache] {run}", flush=True)
    rng = np.random.default_rng(run)
    X = random_lists(rng, 1501, 0, 20_000)
    C = X[1][:-1].copy(), X[0][1:].copy()   # the gaps of X
    none = np.zeros(0, np.uint32), np.zeros(0, np.uint32)
    A, F = [], []
    for k in range(24):   # 0 .. 7: X; the others: its gaps, every other one grown into X somewhere
        end = C[1].copy()
        if k % 2:
            end[min(1499, 70 * k)] += 1
        end[:-1] = np.minimum(end[:-1], C[0][1:])
        A.append(X if k < 8 else (C[0], end))
        F.append(X if k % 4 == 1 else none)
    F = [f if f is none or k < 8 else (A[k][0], A[k][1]) for k, f in enumerate(F)]
    a, f = ListSet.from_lists(A), ListSet.from_lists(F)
    L = oracle.Lists(a.off, a.start, a.end, f.off, f.start, f.end)
    h = april.april_lists_from_arrays(GRID, a.off, a.start, a.end, f.off, f.start, f.end)
    V = april.april_lists_to_device(h, april.CODEC_VBYTE)
    every = np.arange(24, dtype=np.uint32)
    table = oracle.filter_pairs(L, L, np.repeat(every, 24), np.tile(every, 24)).reshape(24, 24)
    assert set(np.unique(table)) == {0, 1, 2}
    n = 1_100_000
    r = np.repeat(rng.integers(0, 24, n // run + 1), run)[:n].astype(np.uint32)
    s = rng.integers(0, 24, n).astype(np.uint32)
    bad = rng.random(n) < 0.001
    want = np.where(bad, april.BAD_PAIR, table[r, s])
    r[bad] = 24
    ws = torch.empty(april.april_filter_workspace_size(n, flags=april.WS_DECODE_CACHE), dtype=torch.uint8, device="cuda")
    rt, st = (torch.from_numpy(x.view(np.int32)).cuda() for x in (r, s))
    for kw in ({}, {"flags": april.WS_DECODE_CACHE, "workspace": ws}):
        v = torch.full((n,), 77, dtype=torch.uint8, device="cuda")
        c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
        april.april_filter_pairs(V, V, rt, st, v, c, schedule=april.SCHED_BATCHED, **kw)
        torch.cuda.synchronize()
        assert np.array_equal(v.cpu().numpy(), want)
        assert c.tolist() == np.bincount(want[~bad], minlength=3).tolist()
