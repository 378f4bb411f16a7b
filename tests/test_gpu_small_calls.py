"""Calls of at most 65,536 pairs, whose pairs are dealt out beforehand and whose
verdicts are counted at the end, around the edges: one pair, a pair or two per
XCD, waves with one pair more than others, the largest such call and the
next; counts from verdict arrays at every alignment.  Verdicts and counts are
whole numbers and have to be the oracle's."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402


@pytest.fixture(scope="module")
def tiny():
    R, S, g = synth.configs.tiny()
    LR, LS = (april.april_build_lists(g, p.xy, p.voff, april.STRICT) for p in (R, S))
    r, s = oracle.mbr_join(R, S)
    oR, oS = (oracle.Lists(*h.export()) for h in (LR, LS))
    dR, dS = (april.april_lists_to_device(h) for h in (LR, LS))
    return dR, dS, r, s, oracle.filter_pairs(oR, oS, r, s), oracle.filter_within(oR, oS, r, s)


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 63, 65, 8191, 8192, 8193, 16385, 65535, 65536, 65537])
def test_sizes(tiny, n):
    dR, dS, r, s, want, within = tiny
    at = np.random.default_rng(n).integers(0, len(r), n)
    rt, st = (torch.from_numpy(k[at].view(np.int32)).cuda() for k in (r, s))
    print(f"[small calls] {n} pairs", flush=True)
    buf = torch.full((n + 16,), 77, dtype=torch.uint8, device="cuda")
    ws = torch.empty(april.april_filter_workspace_size(n), dtype=torch.uint8, device="cuda")
    calls = [lambda v, c: april.april_filter_pairs(dR, dS, rt, st, v, c, schedule=april.SCHED_PLAIN),
             lambda v, c: april.april_filter_pairs(dR, dS, rt, st, v, c, schedule=april.SCHED_BATCHED),
             lambda v, c: april.april_filter_pairs(dR, dS, rt, st, v, c, schedule=april.SCHED_BATCHED, workspace=ws),
             lambda v, c: april.april_filter_pairs_static(dR, dS, rt, st, v, c, schedule=april.SCHED_BATCHED),
             lambda v, c: april.april_filter_pairs(dR, dS, rt, st, v, c, schedule=april.SCHED_BATCHED, waves=12),
             lambda v, c: april.april_filter_within(dR, dS, rt, st, v, c)]
    for k, call in enumerate(calls):
        ref = (within if k == 5 else want)[at]
        v = buf[k:k + n]   # another alignment each time
        c = torch.full((3,), -1, dtype=torch.int64, device="cuda")
        call(v, c)
        torch.cuda.synchronize()
        assert np.array_equal(v.cpu().numpy(), ref), k
        assert np.array_equal(c.cpu().numpy(), np.bincount(ref, minlength=3)), k
        assert int(buf[k + n]) == 77 or k + n >= n + 16
        buf.fill_(77)


def test_captured(tiny):
    """A small call in a graph, replayed with eager work in between."""
    dR, dS, r, s, want, _ = tiny
    rt, st = (torch.from_numpy(k.view(np.int32)).cuda() for k in (r, s))
    v = torch.empty(len(r), dtype=torch.uint8, device="cuda")
    c = torch.empty(3, dtype=torch.int64, device="cuda")
    ws = torch.empty(april.april_filter_workspace_size(len(r)), dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        april.april_filter_pairs(dR, dS, rt, st, v, c, schedule=april.SCHED_BATCHED, workspace=ws, stream=side)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        april.april_filter_pairs(dR, dS, rt, st, v, c, schedule=april.SCHED_BATCHED, workspace=ws, stream=side)
    for _ in range(4):
        v.fill_(77)
        c.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(v.cpu().numpy(), want)
        assert np.array_equal(c.cpu().numpy(), np.bincount(want, minlength=3))
