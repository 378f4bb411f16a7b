"""Workgroup-bin pairs cut into parts: one overlap planted at the edges of the
parts, in lists that otherwise touch everywhere and overlap nowhere, as an
AA, an AF and an FA overlap, against the oracle.  With 128-interval tiles a
part is at least 2,048 intervals."""

import numpy as np
import pytest

import oracle
from synth.intervals import ListSet, complement_list, random_lists

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402

GRID = (0.0, 0.0, float(1 << 16) * 2.0 ** -30 * (1 << 16), 16)


def lists(A, F):
    a, f = ListSet.from_lists(A), ListSet.from_lists(F)
    o = oracle.Lists(a.off, a.start, a.end, f.off, f.start, f.end)
    h = april.april_lists_from_arrays(GRID, o.offA, o.sA, o.eA, o.offF, o.sF, o.eF, validate=True)
    return o, april.april_lists_to_device(h)


@pytest.mark.parametrize("n", [600, 2047, 4095, 4096, 4097, 8192, 20_001, 70_000])
def test_planted_overlaps(n):
    rng = np.random.default_rng(n)
    print(f"[parts] {n} intervals", flush=True)
    X = random_lists(rng, n + 1, 0, 12 * n + 64)
    C = complement_list(*X)
    none = (np.zeros(0, np.uint32), np.zeros(0, np.uint32))
    at = {0, 1, n - 1}
    for of in range(2, 33):
        for part in range(1, of):
            i = (n + 1) * part // of
            at |= {i - 1, i, min(i + 1, n - 1)} if part in (1, of // 2, of - 1) else set()
    at = sorted(k for k in at if 0 <= k < n)
    at = [at[k] for k in np.unique(np.linspace(0, len(at) - 1, 40).astype(int))]
    A, F = [C, C], [none, C]
    for t in at:
        end = C[1].copy()
        end[t] += 1          # the gap now overlaps the interval behind it
        A += [(C[0], end), (C[0], end)]
        F += [none, (C[0][t:t + 1], end[t:t + 1])]
    oS, dS = lists(A, F)
    r, s = np.zeros(len(A), np.uint32), np.arange(len(A), dtype=np.uint32)
    for XF in (none, X):
        oR, dR = lists([X], [XF])
        for (oa, da), (ob, db), (i, j) in (((oR, dR), (oS, dS), (r, s)), ((oS, dS), (oR, dR), (s, r))):
            want = oracle.filter_pairs(oa, ob, i, j)
            v = torch.full((len(i),), 77, dtype=torch.uint8, device="cuda")
            c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
            it, jt = (torch.from_numpy(k.view(np.int32)).cuda() for k in (i, j))
            april.april_filter_pairs(da, db, it, jt, v, c, schedule=april.SCHED_BATCHED, tile=128, wg_min=1)
            torch.cuda.synchronize()
            assert np.array_equal(v.cpu().numpy(), want)
            assert np.array_equal(c.cpu().numpy(), np.bincount(want, minlength=3))
            assert len(np.unique(want)) >= 2


@pytest.mark.parametrize("n", [120_000, 140_000, 600_000, 1_000_000, 1_200_000])
def test_full_queues(n):
    """Every pair is queued: queues without and with room for the parts'
    answers, and ones that overflow."""
    rng = np.random.default_rng(n)
    print(f"[parts] {n} pairs", flush=True)
    none = (np.zeros(0, np.uint32), np.zeros(0, np.uint32))
    A = []
    for _ in range(20):
        s, e = random_lists(rng, 520, 100, 8000)
        A.append((np.append(np.uint32(50), s), np.append(np.uint32(60), e)))
    _, D = lists(A, [none] * 20)
    r, s = (torch.from_numpy(rng.integers(0, 20, n).astype(np.int32)).cuda() for _ in range(2))
    v = torch.full((n,), 77, dtype=torch.uint8, device="cuda")
    c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    april.april_filter_pairs(D, D, r, s, v, c, schedule=april.SCHED_BATCHED, tile=128, wg_min=1)
    torch.cuda.synchronize()
    assert int((v != april.INDECISIVE).sum()) == 0
    assert c.tolist() == [0, 0, n]
