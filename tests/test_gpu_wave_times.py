"""APRIL_WAVE_TIMES where a call takes more kernels than one: the wave kernel's
latest end less its earliest is that kernel's tail, so it is a small part of a
call whose kernels run one after another for long."""

import numpy as np
import pytest

from synth.intervals import ListSet, random_lists

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402

GRID = (0.0, 0.0, float(1 << 16) * 2.0 ** -30 * (1 << 16), 16)


def times(D, r, s, **kw):
    ws = torch.zeros(april.april_filter_workspace_size(len(r)), dtype=torch.uint8, device="cuda")
    v = torch.empty(len(r), dtype=torch.uint8, device="cuda")
    c = torch.zeros(3, dtype=torch.int64, device="cuda")
    for _ in range(2):
        april.april_filter_pairs(D, D, r, s, v, c, schedule=april.SCHED_BATCHED, flags=april.WAVE_TIMES, workspace=ws,
                                 **kw)
        torch.cuda.synchronize()
    at = april.WAVE_TIMES_OFFSET
    return c.tolist(), [int(x) for x in ws[at:at + 40].cpu().numpy().view(np.uint64)]


# F-lists as A-lists: decided by screening but for 1 pair in 16; empty: all open
@pytest.mark.parametrize("share, pairs", [(1 / 16, 5 << 23), (1.0, 1 << 22), (1.0, 3 << 23)])
def test_tail(share, pairs):
    print(f"[times] {share} {pairs}", flush=True)
    rng = np.random.default_rng(pairs)
    A = [random_lists(rng, 200, 0, 3200) for _ in range(64)]
    a = ListSet.from_lists(A)
    F = A if share < 1 else [(np.zeros(0, np.uint32), np.zeros(0, np.uint32))] * 64
    if share < 1:   # objects 60 .. 63 meet all in A only
        F = F[:60] + [(np.zeros(0, np.uint32), np.zeros(0, np.uint32))] * 4
    f = ListSet.from_lists(F)
    D = april.april_lists_to_device(april.april_lists_from_arrays(GRID, a.off, a.start, a.end, f.off, f.start, f.end))
    s = torch.randint(0, 64, (pairs,), dtype=torch.int32, device="cuda")
    r = torch.where(s >= 60, s, torch.randint(0, 60, (pairs,), dtype=torch.int32, device="cuda"))
    counts, (start, first, last, wg_first, wg_last) = times(D, r, s)
    assert counts[2] == (pairs if share == 1 else int((s >= 60).sum()))
    assert start < first <= last and wg_first == 2 ** 64 - 1 and wg_last == 0
    assert last - first < 0.4 * (last - start)
