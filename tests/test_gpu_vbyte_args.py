"""Compressed filter calls that are refused write nothing."""

import numpy as np
import pytest

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
