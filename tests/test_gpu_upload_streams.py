"""Collections that were uploaded or built on one stream, used at once on
another: lists, cells and summaries are complete when the call returns."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402


@pytest.fixture(scope="module")
def data():
    R, S, g = synth.configs.tiny()
    r, s = oracle.mbr_join(R, S)
    times = 9000 // len(r) + 1   # enough pairs to be screened
    r, s = np.tile(r, times), np.tile(s, times)
    hR, hS = (april.april_build_lists(g, P.xy, P.voff, april.STRICT) for P in (R, S))
    cells = april.april_build_cells(g, S.xy, S.voff, april.STRICT)
    LR, LS = oracle.build_lists(g, R), oracle.build_lists(g, S)
    want = {"pairs": oracle.filter_pairs(LR, LS, r, s),
            "lines": oracle.filter_linestrings(LR, oracle.Cells(*cells.export()), r, s)}
    return R, g, hR, hS, cells, r, s, want


@pytest.mark.parametrize("codec", ["raw", "vbyte", "built"])
def test_other_stream(data, codec):
    R, g, hR, hS, cells, r, s, want = data
    print(f"[streams] {codec}", flush=True)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    rt, st = (torch.from_numpy(k.view(np.int32)).cuda() for k in (r, s))
    busy = torch.randn(4096, 4096, device="cuda")
    v = {k: torch.full((len(r),), 77, dtype=torch.uint8, device="cuda") for k in want}
    torch.cuda.synchronize()
    for _ in range(3):
        with torch.cuda.stream(one):
            for _ in range(20):   # some milliseconds of work before the uploads
                busy = busy @ busy * 1e-4
        if codec == "built":
            dR = april.april_build_lists_gpu(g, R.xy, R.voff, april.STRICT, stream=one)
        else:
            dR = april.april_lists_to_device(hR, april.CODEC_RAW if codec == "raw" else april.CODEC_VBYTE, stream=one)
        dS = april.april_lists_to_device(hS, april.CODEC_VBYTE if codec == "vbyte" else april.CODEC_RAW, stream=one)
        dC = april.april_cells_to_device(cells, stream=one)
        april.april_filter_pairs(dR, dS, rt, st, v["pairs"], schedule=april.SCHED_BATCHED, stream=two)
        if codec != "vbyte":
            april.april_filter_linestrings(dR, dC, rt, st, v["lines"], stream=two)
        torch.cuda.synchronize()
        for k in want:
            if codec != "vbyte" or k == "pairs":
                assert np.array_equal(v[k].cpu().numpy(), want[k]), k
