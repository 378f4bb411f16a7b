"""Screening against the oracle's Alg. 2, at the sizes where it can go wrong:
summaries of 32 + 32 intervals, tables of 64 to 512 entries, coarse tables of
128 from 512 intervals on, lists over 2,048 intervals (another kernel), values
that are all equal (the selection's ties), and F-lists outside their A-lists,
which unvalidated lists may hold.  Verdicts and counts are whole numbers and
have to be equal."""

import numpy as np
import pytest

import oracle
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
