"""Refinement of polygons with many edges, by boxes of 64 edges, against the
oracle's exact geometry: vertex counts at the edges of a box, of 64 boxes and
of the rule that takes this path (more than 2^16 edge pairs), against small and
large partners, crossing, nested without contact, and apart.  The answers are
whole numbers and have to be equal."""

import numpy as np
import pytest

import oracle
from synth.polygons import PolygonSet, star_polygons

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402


def refine(R, S, r, s):
    PR, PS = (april.april_polys_to_device(p.xy, p.voff, april.STRICT) for p in (R, S))
    out = torch.full((len(r),), 77, dtype=torch.uint8, device="cuda")
    cnt = torch.full((2,), -1, dtype=torch.int64, device="cuda")
    april.april_refine_pairs(PR, PS, torch.from_numpy(r.astype(np.int32)).cuda(),
                             torch.from_numpy(s.astype(np.int32)).cuda(), out, counts=cnt)
    torch.cuda.synchronize()
    return out.cpu().numpy(), cnt.cpu().numpy()


@pytest.mark.parametrize("sizes", [(255, 256, 257, 319, 320, 321), (12, 64, 65, 300, 1000), (4095, 4096, 4097, 4161),
                                   (8, 8191, 8193)])
def test_box_edges(sizes):
    rng = np.random.default_rng(sum(sizes))
    nv = np.array(sizes * (12 if max(sizes) < 4000 else 2))
    n = len(nv)
    print(f"[refine boxes] {sizes}", flush=True)

    def stars(radius):
        return star_polygons(rng, 0.5 + 0.002 * rng.standard_normal((n, 2)), radius, nv, a=0.1)

    R, S = stars(rng.uniform(0.0005, 0.003, n)), stars(rng.uniform(0.0002, 0.003, n))
    r, s = (k.ravel() for k in np.meshgrid(np.arange(n), np.arange(n), indexing="ij"))
    want = np.array([int(oracle.polygons_intersect(R.polygon(int(a)), S.polygon(int(b)))) for a, b in zip(r, s)])
    assert 0 < want.sum() < len(want)
    got, cnt = refine(R, S, r, s)
    assert np.array_equal(got, want)
    assert cnt.tolist() == [int(want.sum()), len(want)]
    got, _ = refine(S, R, s, r)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("inner,outer", [(20, 300), (300, 20), (300, 5000), (5000, 300), (4096, 4096)])
def test_nested_without_contact(inner, outer):
    """Only the crossing counts decide, over boxes that the ray meets."""
    rng = np.random.default_rng(inner + outer)
    n = 10
    c = 0.5 + 0.01 * rng.standard_normal((n, 2))
    big = star_polygons(rng, c, np.full(n, 0.002), np.full(n, outer), a=0.1)
    far = star_polygons(rng, c + [0.00165, 0.00165], np.full(n, 0.0003), np.full(n, inner), a=0.1)
    small = star_polygons(rng, c + rng.uniform(-3e-4, 3e-4, (n, 2)), np.full(n, 0.0004), np.full(n, inner), a=0.1)
    k = np.arange(n)
    for other in (small, far):   # inside; outside, in a corner of the box
        want = np.array([int(oracle.polygons_intersect(big.polygon(i), other.polygon(i))) for i in k])
        assert want.all() if other is small else not want.any()
        assert np.array_equal(refine(big, other, k, k)[0], want)
        assert np.array_equal(refine(other, big, k, k)[0], want)
    assert isinstance(big, PolygonSet)
