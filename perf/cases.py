"""The work that this framework is timed on: seeded cases and one pass over each.

listed() names the cases, draw() gives more of the same ranges, prepare() makes
what a program holds before the call (device lists, polygons, pair ids, a
server), run() is one pass through the public entry points of
paper_2307_01716_amd.april, work() the bytes that a pass cannot do without.

Every collection is drawn like the repository's workloads: star polygons on
the 2^-30 lattice, centres from a Gaussian mixture that both sides share,
log-normal radii and vertex counts ("scale"); with some polygons of
20k-100k vertices on each side ("skewed"); with objects sixteen times as large
against the grid, as one partition of a 16 x 16 partitioned join sees them
("zoom"); 8-64 vertices on a 2^10 grid ("tiny"); or polygons of 1k-20k
vertices ("complex").  Candidate pairs come from the library's MBR join.

Every output is a whole number (verdicts, counts, ids), so there is no
rounding to compare with and exact() has nothing to say.
"""

import math

import numpy as np
import torch

from paper_2307_01716_amd import april

LATTICE = 2.0 ** -30

# (x0, y0, side) of the square data space.  Objects of the scale workload reach
# 0.02 over the unit square, the larger ones 0.1.
NEAR = (-1.0 / 32, -1.0 / 32, 1.0 + 1.0 / 16)
WIDE = (-1.0 / 8, -1.0 / 8, 1.25)


# ------------------------------------------------------------------ cases

def listed():
    return [
        # The smallest call: a thousand small polygons a side on a coarse grid,
        # library defaults (plain schedule), counts asked for.  Launches and
        # host time are what it costs.
        {"name": "plain_tiny", "kind": "filter", "data": "tiny", "n": 1000, "schedule": "plain", "codec": "raw"},
        # The default call on an ordinary join: one wavefront per pair.
        {"name": "plain_100k", "kind": "filter", "data": "scale", "n": 100_000, "schedule": "plain", "codec": "raw"},
        # The at-scale join, 200k x 200k at grid order 16, about 4.7M pairs, on
        # the schedule that large joins use.
        {"name": "batched_200k", "kind": "filter", "data": "scale", "n": 200_000, "schedule": "batched",
         "codec": "raw"},
        # Heavy tail of complex objects: long lists against short ones, and
        # pairs of two long ones.
        {"name": "batched_skewed", "kind": "filter", "data": "skewed", "n": 40_000, "n_large": 300,
         "schedule": "batched", "codec": "raw"},
        # One partition's worth of a partitioned join: lists of thousands of
        # intervals, raw, ...
        {"name": "batched_zoom", "kind": "filter", "data": "zoom", "n": 10_000, "schedule": "batched", "codec": "raw"},
        # ... and delta + VByte compressed.
        {"name": "vbyte_zoom", "kind": "filter", "data": "zoom", "n": 8_000, "schedule": "batched", "codec": "vbyte"},
        # The query variants: containment, and polygons against linestrings.
        {"name": "within_100k", "kind": "within", "data": "scale", "n": 100_000},
        {"name": "lines_100k", "kind": "lines", "data": "scale", "n": 100_000},
        # A whole join: filter, then exact refinement of what it leaves open.
        {"name": "join_100k", "kind": "join", "data": "scale", "n": 100_000},
        # Exact refinement of every candidate pair of large polygons.
        {"name": "refine_complex", "kind": "refine", "data": "complex", "n": 300},
        # New polygons arrive: their lists are built on the GPU and filtered
        # against a resident collection.
        {"name": "build_50k", "kind": "build", "data": "scale", "n": 50_000},
        # Served selection queries, all offered at once (saturation).
        {"name": "serve_400", "kind": "serve", "data": "scale", "n": 100_000, "queries": 400},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain_tiny", "plain", "batched", "skewed", "zoom", "vbyte", "within", "lines", "join",
                       "refine", "build", "serve"])
    if kind == "plain_tiny":
        return {"kind": "filter", "data": "tiny", "n": _log_int(rng, 60, 4000),
                "schedule": rng.choice(["plain", "batched"]), "codec": "raw"}
    if kind in ("plain", "batched"):
        return {"kind": "filter", "data": "scale", "n": _log_int(rng, 1500, 190_000), "schedule": kind, "codec": "raw"}
    if kind == "skewed":
        return {"kind": "filter", "data": "skewed", "n": _log_int(rng, 2000, 40_000),
                "n_large": _log_int(rng, 20, 300), "schedule": "batched", "codec": "raw"}
    if kind in ("zoom", "vbyte"):
        return {"kind": "filter", "data": "zoom", "n": _log_int(rng, 300, 8000), "schedule": "batched",
                "codec": "vbyte" if kind == "vbyte" else "raw"}
    if kind in ("within", "lines", "join"):
        return {"kind": kind, "data": "scale", "n": _log_int(rng, 2000, 120_000)}
    if kind == "refine":
        return {"kind": "refine", "data": rng.choice(["complex", "complex", "scale"]), "n": _log_int(rng, 60, 300)}
    if kind == "build":
        return {"kind": "build", "data": "scale", "n": _log_int(rng, 300, 60_000)}
    return {"kind": "serve", "data": "scale", "n": _log_int(rng, 5000, 100_000), "queries": _log_int(rng, 8, 400)}


# ----------------------------------------------------------------- inputs

class _Draws:
    """Random numbers of one collection, made on the GPU."""

    def __init__(self, *seed):
        mixed = 0
        for s in seed:
            mixed = (mixed * 1_000_003 + int(s) + 12345) % (1 << 62)
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.gen = torch.Generator(device=self.dev).manual_seed(mixed)

    def uniform(self, lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, generator=self.gen, device=self.dev, dtype=torch.float64)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.gen, device=self.dev, dtype=torch.float64)

    def pick(self, n, weights):
        return torch.multinomial(weights, n, replacement=True, generator=self.gen)


def _snap(v):
    return torch.round(v * 2.0 ** 30) * LATTICE


def _mixture(d, n):
    """Centres from the 64-component Gaussian mixture that all collections share."""
    m = np.random.default_rng(2000)
    means, sigma, weights = (torch.from_numpy(v).to(d.dev) for v in (
        m.uniform(0.05, 0.95, (64, 2)), m.uniform(0.012, 0.03, 64), m.uniform(0.5, 1.5, 64)))
    comp = d.pick(n, weights)
    return (means[comp] + sigma[comp, None] * d.normal(n, 2)).clamp(0.0, 1.0)


def _stars(d, centres, radii, nv, a):
    """Star polygons: vertex m at a jittered angle, between (1 - a) r and r from the centre."""
    off = torch.zeros(len(nv) + 1, dtype=torch.int64, device=d.dev)
    torch.cumsum(nv, 0, out=off[1:])
    seg = torch.repeat_interleave(torch.arange(len(nv), device=d.dev), nv)
    m = torch.arange(len(seg), device=d.dev) - off[seg]
    theta = 2.0 * math.pi * (m + 0.5 + 0.8 * (d.uniform(0, 1, len(seg)) - 0.5)) / nv[seg]
    rho = radii[seg] * (1.0 - a[seg] * d.uniform(0, 1, len(seg)))
    at = _snap(centres)[seg]
    xy = _snap(torch.stack([at[:, 0] + rho * torch.cos(theta), at[:, 1] + rho * torch.sin(theta)], 1))
    return xy.cpu().numpy(), off.cpu().numpy()


def _log_normal(d, n, median, sigma, lo, hi):
    return torch.exp(math.log(median) + sigma * d.normal(n)).clamp(lo, hi)


def _polygons(case, seed, side, n=None):
    """(xy, voff) of one side of a case, on the host."""
    d, data, n = _Draws(seed, side), case["data"], int(n or case["n"])
    if data == "tiny":
        return _stars(d, d.uniform(0, 1, n, 2), d.uniform(0.002, 0.02, n), d.uniform(8, 65, n).long(),
                      torch.full((n,), 0.3, device=d.dev, dtype=torch.float64))
    if data == "complex":
        return _stars(d, _mixture(d, n), d.uniform(0.02, 0.1, n), d.uniform(1000, 20_001, n).long(),
                      torch.full((n,), 0.02, device=d.dev, dtype=torch.float64))
    zoom = 16.0 if data == "zoom" else 1.0
    centres = d.uniform(0, 1, n, 2) if data == "zoom" else _mixture(d, n)
    radii = _log_normal(d, n, 0.001 * zoom, 0.6, 2e-4 * zoom, min(0.1, 0.02 * zoom))
    nv = torch.round(_log_normal(d, n, 30.0, 0.7, 8, 5000)).long()
    a = torch.full((n,), 0.3, device=d.dev, dtype=torch.float64)
    if data == "skewed":
        k = int(case["n_large"])
        centres = torch.cat([centres, _mixture(d, k)])
        radii = torch.cat([radii, d.uniform(0.02, 0.1, k)])
        nv = torch.cat([nv, d.uniform(20_000, 100_001, k).long()])
        a = torch.cat([a, torch.full((k,), 0.02, device=d.dev, dtype=torch.float64)])
    return _stars(d, centres, radii, nv, a)


def _walks(seed, n):
    """Random-walk linestrings: log-normal vertex counts (median 12) and steps (median 3e-4)."""
    d = _Draws(seed, 9)
    k = torch.round(_log_normal(d, n, 12.0, 0.8, 2, 200)).long()
    off = torch.zeros(n + 1, dtype=torch.int64, device=d.dev)
    torch.cumsum(k, 0, out=off[1:])
    seg = torch.repeat_interleave(torch.arange(n, device=d.dev), k)
    ang, step = d.uniform(0, 2 * math.pi, len(seg)), _log_normal(d, len(seg), 3e-4, 0.7, 0, 0.02)
    c = torch.cumsum(torch.stack([torch.cos(ang) * step, torch.sin(ang) * step], 1), 0)
    xy = _snap((_mixture(d, n)[seg] + c - c[off[:-1]][seg]).clamp(-0.02, 1.02))
    return xy.cpu().numpy(), off.cpu().numpy()


def _queries(seed, n):
    """Query polygons of 10 to 10^4 vertices, radius 5e-4 to 0.05, both log-uniform."""
    d = _Draws(seed, 3)
    radii = torch.exp(d.uniform(math.log(5e-4), math.log(0.05), n))
    nv = torch.round(torch.exp(d.uniform(math.log(10.0), math.log(1e4), n))).long()
    return _stars(d, _mixture(d, n), radii, nv, torch.full((n,), 0.3, device=d.dev, dtype=torch.float64))


def _boxes(xy, voff):
    at = voff[:-1]
    return np.stack([np.minimum.reduceat(xy[:, 0], at), np.minimum.reduceat(xy[:, 1], at),
                     np.maximum.reduceat(xy[:, 0], at), np.maximum.reduceat(xy[:, 1], at)], 1)


def _grid(case):
    space = NEAR if case["data"] in ("tiny", "scale") and case["kind"] != "serve" else WIDE
    return space + (10 if case["data"] == "tiny" else 16,)


def _pairs(case, R, S):
    """Candidate pairs of the MBR join: a batch of a fixed number of them (some
    twice where a seed gives fewer), as a program with buffers of its own takes them."""
    r, s = april.april_mbr_join(_boxes(*R), _boxes(*S))
    n = pairs_of(case)
    r, s = np.resize(r, n), np.resize(s, n)
    return torch.from_numpy(r.view(np.int32)).cuda(), torch.from_numpy(s.view(np.int32)).cuda()


def _lists(case, grid, P):
    dev = april.april_build_lists_gpu(grid, P[0], P[1], april.STRICT)
    if case.get("codec") != "vbyte":
        return dev
    host = april.april_lists_download(dev)
    dev.free()
    return april.april_lists_to_device(host, april.CODEC_VBYTE)


# --------------------------------------------------------- prepare and run

def prepare(case, seed):
    kind, grid = case["kind"], _grid(case)
    R = _polygons(case, seed, 1)
    st = {"kind": kind}
    if kind == "serve":
        st["server"] = april.Server(_lists(case, grid, R), _boxes(*R))
        xy, off = _queries(seed, int(case["queries"]))
        # about three times the answers that the queries have on average
        st["room"] = int(int(case["n"]) * (0.01 * int(case["queries"]) + 0.3))
        st["queries"] = [xy[off[k]:off[k + 1]] for k in range(len(off) - 1)]
        return st
    S = _walks(seed, int(case["n"])) if kind == "lines" else _polygons(case, seed, 2)
    st["r"], st["s"] = _pairs(case, R, S)
    n = st["r"].numel()
    st["verdict"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    st["counts"] = torch.zeros(3, dtype=torch.int64, device="cuda")
    if kind in ("join", "refine"):
        st["PR"] = april.april_polys_to_device(*R, april.STRICT)
        st["PS"] = april.april_polys_to_device(*S, april.STRICT)
        st["meet"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        st["tested"] = torch.zeros(2, dtype=torch.int64, device="cuda")
    if kind == "build":
        st["grid"], st["xy"], st["voff"] = grid, R[0], R[1]
    elif kind != "refine":
        st["R"] = _lists(case, grid, R)
    if kind == "lines":
        st["S"] = april.april_cells_to_device(april.april_build_cells(grid, *S, april.STRICT))
    elif kind != "refine":
        st["S"] = _lists(case, grid, S)
    plain = case.get("schedule") == "plain"
    st["schedule"] = april.SCHED_PLAIN if plain else april.SCHED_BATCHED
    return st


def run(st):
    kind = st["kind"]
    if kind == "serve":
        srv = st["server"]
        tickets = [srv.submit(q) for q in st["queries"]]
        found = []
        for t in tickets:
            found.append(srv.wait(t, 600))
            srv.release(t)
        # the answers one after another, in arrays of a fixed size
        at = np.cumsum([0] + [len(f.s_ids) for f in found])
        ids, verdict = np.zeros(st["room"], np.uint32), np.zeros(st["room"], np.uint8)
        for f, k in zip(found, at):
            m = max(0, min(len(f.s_ids), st["room"] - int(k)))
            ids[k:k + m], verdict[k:k + m] = f.s_ids[:m], f.verdict[:m]
        return {"at": at, "ids": ids, "verdict": verdict}
    if kind == "refine":
        april.april_refine_pairs(st["PR"], st["PS"], st["r"], st["s"], st["meet"], counts=st["tested"])
        return {"meet": st["meet"], "tested": st["tested"]}
    if kind == "within":
        april.april_filter_within(st["R"], st["S"], st["r"], st["s"], st["verdict"], st["counts"])
    elif kind == "lines":
        april.april_filter_linestrings(st["R"], st["S"], st["r"], st["s"], st["verdict"], st["counts"])
    elif kind == "build":
        lists = april.april_build_lists_gpu(st["grid"], st["xy"], st["voff"], april.STRICT)
        april.april_filter_pairs(lists, st["S"], st["r"], st["s"], st["verdict"], st["counts"],
                                 schedule=st["schedule"])
        info = lists.info()
        lists.free()
        return {"verdict": st["verdict"], "counts": st["counts"], "n_a": int(info.n_a), "n_f": int(info.n_f)}
    else:
        april.april_filter_pairs(st["R"], st["S"], st["r"], st["s"], st["verdict"], st["counts"],
                                 schedule=st["schedule"])
    if kind == "join":
        april.april_refine_pairs(st["PR"], st["PS"], st["r"], st["s"], st["meet"], verdict=st["verdict"],
                                 counts=st["tested"])
        return {"verdict": st["verdict"], "counts": st["counts"], "meet": st["meet"], "tested": st["tested"]}
    return {"verdict": st["verdict"], "counts": st["counts"]}


# -------------------------------------------------------------------- work

# Means of the generators above, from their host-built lists and MBR joins:
# vertices and list intervals (A and F together) of one object, and candidate
# pairs as a share of n * n (a little below the mean, which seeds vary about).
VERTICES = {"tiny": 36.0, "scale": 38.0, "zoom": 38.0, "complex": 10_500.0}
INTERVALS = {"tiny": 42.0, "scale": 327.0, "zoom": 4500.0}
LARGE_INTERVALS = 137_000.0
PAIR_SHARE = {"tiny": 1.65e-3, "scale": 1.13e-4, "zoom": 5.4e-3, "complex": 7.8e-2}
SMALL_LARGE_SHARE, LARGE_SHARE = 0.029, 0.08
RUNS_PER_LINE, LINE_PAIR_SHARE = 209.0, 8.2e-5
VBYTE_RATIO = 3.4      # raw bytes per compressed byte


def pairs_of(case):
    """Candidate pairs in a pass."""
    n, data = float(case["n"]), case["data"]
    pairs = n * n * (LINE_PAIR_SHARE if case["kind"] == "lines" else PAIR_SHARE.get(data, PAIR_SHARE["scale"]))
    if data == "skewed":
        k = float(case["n_large"])
        pairs += 2 * n * k * SMALL_LARGE_SHARE + k * k * LARGE_SHARE
    return max(1, int(pairs))


def work(case):
    """Lists, pair ids (or polygons) read once, verdicts and counts written once."""
    kind, data, n = case["kind"], case["data"], float(case["n"])
    if kind == "serve":
        q = float(case["queries"])
        return {"bytes": q * 16 * 1450 + 8 * INTERVALS["scale"] * n + q * 5 * 3600 * n / 1e6, "flops": 0}
    pairs = pairs_of(case)
    objects = 8 * n * INTERVALS.get(data, INTERVALS["scale"])
    if data == "skewed":
        objects += 8 * float(case["n_large"]) * LARGE_INTERVALS
    if case.get("codec") == "vbyte":
        objects /= VBYTE_RATIO
    polygons = 16 * n * VERTICES.get(data, VERTICES["scale"])
    ids = pairs * 8 + pairs + 24
    if kind == "refine":
        return {"bytes": 2 * polygons + ids, "flops": 0}
    if kind == "build":
        return {"bytes": polygons + 2 * objects + ids, "flops": 0}
    if kind == "lines":
        return {"bytes": objects + 8 * n * RUNS_PER_LINE + ids, "flops": 0}
    if kind == "join":
        return {"bytes": 2 * objects + 0.02 * 2 * polygons + ids + 2 * pairs, "flops": 0}
    return {"bytes": 2 * objects + ids, "flops": 0}


def exact(case, seed):
    """Outputs are whole numbers only: they are equal or they are wrong."""
    return None
