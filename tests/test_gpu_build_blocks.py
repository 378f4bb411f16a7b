"""The GPU list builder at the edges of its blocks of 64 x 64 cells, against the
host builder, bit for bit: grids smaller than a block, of one block and of
many; polygons inside a block, along its lines and across its corners,
larger than several blocks; vertices on cell lines, corners and centres;
vertex counts at the edges of the boxes of 64 edges; 64-bit and 128-bit
arithmetic."""

import numpy as np
import pytest

from synth.polygons import LATTICE, PolygonSet

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2307_01716_amd import april  # noqa: E402


def stars(rng, centres, radii, nv, quantum):
    """Star polygons with vertices rounded to `quantum` lattice units (lattice units throughout)."""
    xy = []
    for c, r, n in zip(centres, radii, nv):
        th = 2 * np.pi * (np.arange(n) + 0.5 + 0.6 * (rng.random(n) - 0.5)) / n
        rho = r * (1 - 0.3 * rng.random(n))
        p = np.stack([c[0] + rho * np.cos(th), c[1] + rho * np.sin(th)], 1)
        xy.append(np.round(p / quantum) * quantum)
    voff = np.zeros(len(xy) + 1, np.int64)
    np.cumsum([len(p) for p in xy], out=voff[1:])
    return PolygonSet(np.concatenate(xy) * LATTICE, voff)


def check(grid, ps, what):
    print(f"[build blocks] {what}: {len(ps)} polygons, {len(ps.xy)} vertices", flush=True)
    host = april.april_build_lists(grid, ps.xy, ps.voff, april.STRICT).export()
    dev = april.april_build_lists_gpu(grid, ps.xy, ps.voff, april.STRICT)
    got = april.april_lists_download(dev).export()
    for name, x, y in zip(("offA", "sA", "eA", "offF", "sF", "eF"), host, got):
        assert np.array_equal(x, y), (what, name)


@pytest.mark.parametrize("w", [8, 1 << 14, 1 << 23])
@pytest.mark.parametrize("order", [3, 5, 6, 7, 9, 12, 16])
def test_orders(order, w):
    if w > 1 << 14 and order > 9:
        pytest.skip("beyond the coordinates that polygons may have")
    rng = np.random.default_rng(order * 100 + w % 97)
    n, cells = 150, 1 << order
    grid = (0.0, 0.0, float(w * cells) * LATTICE, order)
    top = min(cells / 2 - 1.9, 200.0)   # cells
    for quantum, what in ((w // 2, "on lines and centres"), (max(1, w // 4), "quarters"), (1, "anywhere")):
        r = np.exp(rng.uniform(np.log(min(1.5, top)), np.log(top), n))
        c = rng.uniform((r + 1.7)[:, None], (cells - 1.7 - r)[:, None], (n, 2))
        if cells > 128:   # half of them around corners of blocks
            k = n // 2
            r[:k] = np.minimum(r[:k], 50)
            c[:k] = 64 * rng.integers(1, cells // 64, (k, 2))
        ok = np.all((c - r[:, None] > 1.6) & (c + r[:, None] < cells - 1.6), axis=1)
        ps = stars(rng, c[ok] * w, r[ok] * w, rng.integers(5, 40, int(ok.sum())), quantum)
        check(grid, ps, f"order {order}, cell {w}, {what}")


@pytest.mark.parametrize("nv", [63, 64, 65, 127, 128, 129, 4095, 4097])
def test_edge_counts(nv):
    rng = np.random.default_rng(nv)
    w, order = 1 << 14, 12
    c = rng.uniform(700, 3300, (5, 2))
    ps = stars(rng, c * w, np.array([3.0, 40, 130, 260, 600]) * w, np.full(5, nv), 1 if nv > 200 else w // 2)
    check((0.0, 0.0, float(w << order) * LATTICE, order), ps, f"{nv} vertices")


def test_shapes_on_block_lines():
    """Squares whose sides run along lines of blocks, a bar through many
    blocks, and one polygon over most of the grid."""
    w, order = 1 << 10, 12
    shapes = []
    for x0, y0, x1, y1 in ((64, 64, 128, 128), (63, 63, 64, 64), (64, 128, 65, 192), (100, 64, 164, 65),
                           (60, 60, 70, 4000), (2, 2000, 4093, 2001), (2, 2, 4094, 4094)):
        shapes.append(np.array([[x0, y0], [x1, y0], [x1, y1], [x0, y1]], float))
    shapes.append(np.array([[64, 64], [128.5, 192], [64, 320], [63.5, 192]]))
    voff = 4 * np.arange(len(shapes) + 1)
    check((0.0, 0.0, float(w << order) * LATTICE, order), PolygonSet(np.concatenate(shapes) * w * LATTICE, voff),
          "shapes on block lines")


def test_groups_of_polygons():
    """70 polygons over nearly all of the finest grid: 73 million blocks, more
    than are worked on at once."""
    rng = np.random.default_rng(70)
    w, order = 1 << 14, 16
    far = (1 << order) - 3
    shapes = []
    for _ in range(70):
        lo, hi = rng.uniform(2, 60, (2, 2)), rng.uniform(far - 60, far, (2, 2))
        shapes.append(np.round(np.array([[lo[0, 0], lo[0, 1]], [hi[0, 0], lo[1, 1]], [hi[1, 0], hi[1, 1]],
                                         [lo[1, 0], hi[0, 1]]]) * w))
    check((0.0, 0.0, float(w << order) * LATTICE, order),
          PolygonSet(np.concatenate(shapes) * LATTICE, 4 * np.arange(71)), "two groups")
