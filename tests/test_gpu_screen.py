"""Screening against the oracle's Alg. 2, at the sizes where it can go wrong:
summaries of 32 + 32 intervals, tables of 64 to 512 entries, coarse tables of
128 from 512 intervals on, lists over 2,048 intervals (another kernel), values
that are all equal (the selection's ties), and F-lists outside their A-lists,
which unvalidated lists may hold.  Verdicts and counts are whole numbers and
have to be equal."""

import numpy as np
import pytest

import oracle
from synth.grid import Grid
from synth.intervals import ListSet, random_lists, sub_lists

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402

GRID = (0.0, 0.0, float(1 << 16) * 2.0 ** -30 * (1 << 16), 16)
PAIRS = 9000     # enough to be screened
SIZES = {
    "summary": [0, 1, 2, 31, 32, 33, 34, 63, 64, 65],
    "tables": [62, 63, 64, 126, 127, 128, 129, 255, 256, 257],
    "coarse": [500, 511, 512, 513, 640, 1023, 1024, 1025],
    "long": [1, 40, 700, 2047, 2048, 2049, 5000, 40_000],
}


def lists_of(rng, sizes, n, equal, outside=False):
    """n objects; `equal`: unit intervals at equal gaps, so every value ties."""
    A, F = [], []
    for k in range(n):
        m = int(sizes[k % len(sizes)])
        lo = int(rng.integers(0, 1 << 16)) + (8 if k % 3 else 0) * max(sizes)
        if equal:
            s = (lo + 4 * np.arange(m)).astype(np.uint32)
            a = (s, s + np.uint32(1 + k % 2))
        else:
            a = random_lists(rng, m, lo, lo + 16 * max(m, 4))
        f = sub_lists(rng, *a, p=float(rng.random()))
        if outside:
            f = (f[0] + np.uint32(1 << 20), f[1] + np.uint32(1 << 20))
        A.append(a)
        F.append(f)
    a, f = ListSet.from_lists(A), ListSet.from_lists(F)
    return oracle.Lists(a.off, a.start, a.end, f.off, f.start, f.end)


def upload(L, codec, validate=True):
    h = april.april_lists_from_arrays(GRID, L.offA, L.sA, L.eA, L.offF, L.sF, L.eF, validate=validate)
    return april.april_lists_to_device(h, codec=codec)


def check(LR, LS, r, s, **kw):
    want = oracle.filter_pairs(LR[0], LS[0], r, s)
    v = torch.full((len(r),), 77, dtype=torch.uint8, device="cuda")
    c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    april.april_filter_pairs(LR[1], LS[1], torch.from_numpy(r.view(np.int32)).cuda(),
                             torch.from_numpy(s.view(np.int32)).cuda(), v, c, **kw)
    torch.cuda.synchronize()
    assert np.array_equal(v.cpu().numpy(), want)
    assert np.array_equal(c.cpu().numpy(), np.bincount(want, minlength=3))


@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_edges(sizes, equal):
    rng = np.random.default_rng(len(sizes) + 100 * equal)
    print(f"[screen] {sizes} equal={equal}", flush=True)
    n = 24 if sizes == "long" else 60
    LR, LS = (lists_of(rng, SIZES[sizes], n, equal) for _ in range(2))
    r, s = (rng.integers(0, n, PAIRS).astype(np.uint32) for _ in range(2))
    r.sort()
    for codec in (april.CODEC_RAW, april.CODEC_VBYTE):
        R, S = (LR, upload(LR, codec)), (LS, upload(LS, codec))
        check(R, S, r, s, schedule=april.SCHED_BATCHED)
        if codec == april.CODEC_RAW:
            check(R, S, r, s, schedule=april.SCHED_PLAIN)
            check(S, R, s, r, schedule=april.SCHED_BATCHED, tile=128, wg_min=1)


def test_f_outside_a():
    """The plain schedule takes lists whose F-intervals lie outside A."""
    rng = np.random.default_rng(9)
    LR, LS = (lists_of(rng, [5, 40, 200], 40, False, outside=True) for _ in range(2))
    R, S = (LR, upload(LR, april.CODEC_RAW, False)), (LS, upload(LS, april.CODEC_RAW, False))
    r, s = (rng.integers(0, 40, PAIRS).astype(np.uint32) for _ in range(2))
    check(R, S, r, s, schedule=april.SCHED_PLAIN)


def test_bad_pairs_are_not_counted():
    rng = np.random.default_rng(10)
    LR, LS = (lists_of(rng, [20, 60], 20, False) for _ in range(2))
    R, S = upload(LR, april.CODEC_RAW), upload(LS, april.CODEC_RAW)
    r, s = (rng.integers(0, 20, PAIRS).astype(np.uint32) for _ in range(2))
    want = oracle.filter_pairs(LR, LS, r, s)
    bad = rng.random(PAIRS) < 0.1
    r[bad] = 20 + rng.integers(0, 1 << 20, int(bad.sum())).astype(np.uint32)
    for sched in (april.SCHED_PLAIN, april.SCHED_BATCHED):
        v = torch.zeros(PAIRS, dtype=torch.uint8, device="cuda")
        c = torch.zeros(3, dtype=torch.int64, device="cuda")
        april.april_filter_pairs(R, S, torch.from_numpy(r.view(np.int32)).cuda(),
                                 torch.from_numpy(s.view(np.int32)).cuda(), v, c, schedule=sched)
        got = v.cpu().numpy()
        assert np.array_equal(got, np.where(bad, april.BAD_PAIR, want))
        assert np.array_equal(c.cpu().numpy(), np.bincount(want[~bad], minlength=3))


@pytest.mark.parametrize("sizes", ["tables", "long"])
def test_in_parts(sizes):
    """Calls of more pairs than are screened at a time: the same pairs over and
    over, against one of them by itself."""
    rng = np.random.default_rng(50)
    print(f"[screen] parts {sizes}", flush=True)
    LR, LS = (lists_of(rng, SIZES[sizes], 24, False) for _ in range(2))
    R, S = upload(LR, april.CODEC_RAW), upload(LS, april.CODEC_RAW)
    r, s = (rng.integers(0, 24, PAIRS + 1).astype(np.uint32) for _ in range(2))
    r.sort()
    for fn, want in ((april.april_filter_pairs, oracle.filter_pairs(LR, LS, r, s)),
                     (april.april_filter_within, oracle.filter_within(LR, LS, r, s))):
        times = (1 << 24) // len(r) + 7
        rt, st = (torch.from_numpy(k.view(np.int32)).cuda().repeat(times) for k in (r, s))
        v = torch.full((len(rt),), 77, dtype=torch.uint8, device="cuda")
        c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
        kw = {"schedule": april.SCHED_BATCHED} if fn is april.april_filter_pairs else {}
        fn(R, S, rt, st, v, c, **kw)
        torch.cuda.synchronize()
        assert bool((v.view(times, -1) == torch.from_numpy(want).cuda()).all())
        assert c.tolist() == (np.bincount(want, minlength=3) * times).tolist()


# ------------------------------------------------- within joins, linestrings

def run(fn, *args):
    r, s = args[2:]
    v = torch.full((len(r),), 77, dtype=torch.uint8, device="cuda")
    c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    fn(args[0], args[1], torch.from_numpy(r.view(np.int32)).cuda(), torch.from_numpy(s.view(np.int32)).cuda(), v, c)
    torch.cuda.synchronize()
    return v.cpu().numpy(), c.cpu().numpy()


def inside(rng, fs, fe, n, kind):
    """Up to n intervals, each inside an F-interval; kind 1: and one beyond the
    last, kind 2: and the first one grown over its F-interval's start."""
    take = np.sort(rng.choice(len(fs), min(n, len(fs)), replace=False))
    s, e = fs[take].copy(), fe[take].copy()
    cut = rng.integers(0, e - s)
    keep_end = rng.random(len(s)) < 0.5
    s += np.where(keep_end, cut, 0).astype(np.uint32)
    e -= np.where(keep_end, 0, cut).astype(np.uint32)
    if len(s) and kind == 1:
        s, e = np.append(s, fe[-1] + np.uint32(5)), np.append(e, fe[-1] + np.uint32(6))
    if len(s) and kind == 2:
        s[0] = fs[take[0]] - np.uint32(1)
    return s.astype(np.uint32), e.astype(np.uint32)


def contained(rng, LS, sizes):
    """One object for each of LS: inside its F-intervals, almost so, or not."""
    A, F = [], []
    for k in range(len(LS.offA) - 1):
        f = slice(int(LS.offF[k]), int(LS.offF[k + 1]))
        a = inside(rng, LS.sF[f], LS.eF[f], int(sizes[k % len(sizes)]), k % 3)
        A.append(a)
        F.append(sub_lists(rng, *a, p=0.5))
    a, f = ListSet.from_lists(A), ListSet.from_lists(F)
    return oracle.Lists(a.off, a.start, a.end, f.off, f.start, f.end)


@pytest.mark.parametrize("sizes", list(SIZES))
def test_within(sizes):
    rng = np.random.default_rng(20 + len(sizes))
    print(f"[screen] within {sizes}", flush=True)
    n = 48 if sizes == "long" else 120
    LS = lists_of(rng, SIZES[sizes], n, False)
    LR = contained(rng, LS, SIZES[sizes])
    r = rng.integers(0, n, PAIRS).astype(np.uint32)
    r.sort()
    s = np.where(rng.random(PAIRS) < 0.7, r, rng.integers(0, n, PAIRS)).astype(np.uint32)
    R, S = upload(LR, april.CODEC_RAW), upload(LS, april.CODEC_RAW)
    want = oracle.filter_within(LR, LS, r, s)
    assert set(np.unique(want)) == {0, 1, 2}
    got, counts = run(april.april_filter_within, R, S, r, s)
    assert np.array_equal(got, want)
    assert np.array_equal(counts, np.bincount(want, minlength=3))


def test_within_f_outside_a():
    """Lists whose F-intervals lie outside A: as without screening, which
    calls of few pairs go without."""
    rng = np.random.default_rng(31)
    LR, LS = (lists_of(rng, [5, 40, 200, 600], 40, False, outside=o) for o in (False, True))
    R, S = upload(LR, april.CODEC_RAW), upload(LS, april.CODEC_RAW, False)
    r, s = (rng.integers(0, 40, PAIRS).astype(np.uint32) for _ in range(2))
    parts = [run(april.april_filter_within, R, S, r[i:i + 4500], s[i:i + 4500]) for i in (0, 4500)]
    got, counts = run(april.april_filter_within, R, S, r, s)
    assert np.array_equal(got, np.concatenate([p[0] for p in parts]))
    assert np.array_equal(counts, sum(p[1] for p in parts))


@pytest.mark.parametrize("sizes", list(SIZES))
def test_linestrings(sizes):
    rng = np.random.default_rng(40 + len(sizes))
    print(f"[screen] linestrings {sizes}", flush=True)
    g = Grid(0.0, 0.0, 1.0, 10)
    n, ids = (24 if sizes == "long" else 60), 1 << 20
    A, F = [], []
    for k in range(n):
        m = int(SIZES[sizes][k % len(SIZES[sizes])])
        hi = ids if k % 2 else max(16 * m, ids >> 6)
        lo = int(rng.integers(0, ids - hi + 1)) if hi < ids else 0
        a = random_lists(rng, m, lo, lo + min(hi, ids))
        A.append(a)
        F.append(sub_lists(rng, *a, p=0.3 * float(rng.random())))
    a, f = ListSet.from_lists(A), ListSet.from_lists(F)
    LP = oracle.Lists(a.off, a.start, a.end, f.off, f.start, f.end)
    steps = [1, 2, 20, 40, 60, 100, 300, 4000]
    lines = []
    for k in range(n):
        walk = rng.random(2) + np.cumsum(rng.normal(0, 2.0 ** -9, (steps[k % len(steps)] + 1, 2)), axis=0)
        lines.append(np.round(np.clip(walk, 0.01, 0.99) * 2.0 ** 30) * 2.0 ** -30)
    xy, voff = np.concatenate(lines), np.concatenate([[0], np.cumsum([len(x) for x in lines])]).astype(np.uint64)
    C = april.april_build_cells(g, xy, voff, april.STRICT)
    off, cells = C.export()
    p, l = (rng.integers(0, n, PAIRS).astype(np.uint32) for _ in range(2))
    p.sort()
    want = oracle.filter_linestrings(LP, oracle.Cells(off, cells), p, l)
    assert set(np.unique(want)) == {0, 1, 2}
    h = april.april_lists_from_arrays(g, LP.offA, LP.sA, LP.eA, LP.offF, LP.sF, LP.eF)
    got, counts = run(april.april_filter_linestrings, april.april_lists_to_device(h),
                      april.april_cells_to_device(C), p, l)
    assert np.array_equal(got, want)
    assert np.array_equal(counts, np.bincount(want, minlength=3))


# ----------------------------------------------------- lists of open pairs

@pytest.mark.parametrize("sizes, n", [([3, 40], 70_000), ([3], 900_000), ([600], 300_000), ([600], 600_000),
                                      ([3, 600], 1_000_000)])
def test_open_lists(sizes, n):
    """Every pair is left open (F-lists empty, A-lists that meet): lists that
    hold them all, and lists of either kind that overflow; grids of fewer
    workgroups than there are lists, and of no multiple of them."""
    rng = np.random.default_rng(n)
    print(f"[screen] open {sizes} {n}", flush=True)
    A = [random_lists(rng, sizes[k % len(sizes)], 100, 100 + 16 * sizes[k % len(sizes)]) for k in range(40)]
    a = ListSet.from_lists([(np.append(np.uint32(50), s), np.append(np.uint32(60), e)) for s, e in A])
    off = np.zeros(41, np.uint64)
    none = np.zeros(0, np.uint32)
    L = oracle.Lists(a.off, a.start, a.end, off, none, none)
    D = upload(L, april.CODEC_RAW)
    r, s = (rng.integers(0, 40, n).astype(np.uint32) for _ in range(2))
    rt, st = (torch.from_numpy(k.view(np.int32)).cuda() for k in (r, s))
    calls = [lambda v, c, w=w: april.april_filter_pairs(D, D, rt, st, v, c, schedule=april.SCHED_BATCHED, waves=w)
             for w in (0, 4, 12, 52)]
    calls += [lambda v, c, m=m: april.april_filter_pairs(D, D, rt, st, v, c, schedule=april.SCHED_BATCHED, wg_min=m)
              for m in (1, 0xFFFFFFFF)]   # every pair that can be in the workgroup bin, none
    calls.append(lambda v, c: april.april_filter_within(D, D, rt, st, v, c))
    for k, call in enumerate(calls):
        v = torch.full((n,), 77, dtype=torch.uint8, device="cuda")
        c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
        call(v, c)
        torch.cuda.synchronize()
        assert int((v != april.INDECISIVE).sum()) == 0, k
        assert c.tolist() == [0, 0, n], k


# --------------------------------------------- compressed pairs left open

@pytest.mark.parametrize("holes", [False, True])
@pytest.mark.parametrize("n", [1024, 1025, 1087, 1088, 2049, 6000])
def test_compressed_planted(n, holes):
    """One overlap planted at the edges of blocks of 64 intervals (give or take
    a decoding window) in lists that otherwise touch everywhere, as an AA, an
    AF and an FA overlap.  `holes`: every 100 intervals the other side has 150
    by itself, whose blocks meet nothing of the first one's hull."""
    rng = np.random.default_rng(n + holes)
    print(f"[screen] compressed {n} {holes}", flush=True)
    X = random_lists(rng, n + 1, 0, 12 * n + 64)
    C = X[1][:-1].copy(), X[0][1:].copy()   # the gaps of X
    none = (np.zeros(0, np.uint32), np.zeros(0, np.uint32))
    if holes:
        far = (np.arange(n + 1, dtype=np.uint32) // np.uint32(100)) * np.uint32(400_000)
        C = C[0] + far[:-1], C[1] + far[:-1]
        own = [np.uint32(20 * n + 1000) + np.uint32(400_000) * np.uint32(k) + np.arange(0, 450, 3, dtype=np.uint32)
               for k in range(n // 100 + 1)]
        own = np.concatenate(own)
        X = (np.concatenate([X[0] + far, own]), np.concatenate([X[1] + far, own + np.uint32(1)]))
        o = np.argsort(X[0], kind="stable")
        X = X[0][o].astype(np.uint32), X[1][o].astype(np.uint32)
        keep = np.append(X[1][:-1] <= X[0][1:], True)
        X = X[0][keep], X[1][keep]
    at = sorted({k for b in (0, 64, 128, 192, 512, 1024, n // 2 // 64 * 64, n // 64 * 64, n)
                 for k in (b - 131, b - 65, b - 2, b - 1, b, b + 1, b + 63, b + 129) if 0 <= k < n - 1})
    A, F = [C, C], [none, C]
    for t in at:
        nxt = X[0][np.searchsorted(X[0], C[1][t])]   # the next interval of the other side
        if nxt + 1 > C[0][t + 1]:
            continue
        end = C[1].copy()
        end[t] = nxt + 1
        A += [(C[0], end), (C[0], end)]
        F += [none, (C[0][t:t + 1], end[t:t + 1])]
    for XF in (none, X):
        sides = []
        for a, f in (([X], [XF]), (A, F)):
            a, f = ListSet.from_lists(a), ListSet.from_lists(f)
            L = oracle.Lists(a.off, a.start, a.end, f.off, f.start, f.end)
            sides.append((L, upload(L, april.CODEC_VBYTE)))
        r, s = np.zeros(len(A), np.uint32), np.arange(len(A), dtype=np.uint32)
        assert len(set(oracle.filter_pairs(sides[0][0], sides[1][0], r, s))) > 1
        for tile in (256, 512, 1024):
            check(sides[0], sides[1], r, s, schedule=april.SCHED_BATCHED, tile=tile)
            check(sides[1], sides[0], s, r, schedule=april.SCHED_BATCHED, tile=tile)
