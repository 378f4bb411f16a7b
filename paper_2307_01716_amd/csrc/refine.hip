// Exact refinement of candidate pairs (the step after the intermediate
// filter, Sec. 2): do the two polygons share a point?
//
// Polygons are kept on the device as exact lattice coordinates (multiples
// of 2^-30 as int64), so every predicate is an integer sign.  Two closed
// polygons share a point iff an edge of one meets an edge of the other, or,
// with no boundary contact at all, one lies inside the other -- then any
// vertex of the inner one is strictly inside the outer one.
//
// Layout: one 64-byte record per polygon (first vertex index, vertex count,
// MBR, first vertex) and the vertices as interleaved (x, y) int64 pairs.
//
// Work: waves take G pairs at a time from per-XCD ranges (G = 64 for large
// calls, down to 4 when there are few pairs per wave); a lane reads one pair's
// ids, verdict and both polygon records.  Pairs the filter already decided
// are answered from the verdict; the others are tested one after another by
// the whole wave.  Only edges whose box meets the intersection B of the two
// MBRs can meet (a common point lies in both MBRs), so the others are
// dropped; the kept edges of each side are staged in LDS and tested
// all-pairs, 64 edge pairs per step, with coordinates relative to the lower
// left corner of the MBRs' union: when both polygons span less than 2^31
// lattice units, differences fit in 32 bits and cross products in 64.  The
// ray-crossing counts that decide containment are taken in the same pass
// over the edges.  Wider pairs are marked and left to a second pass, in 128-bit
// arithmetic, and so are pairs of many edges, which go through boxes of 64 of them.
#include <hip/hip_runtime.h>

#include <cmath>
#include <new>

#include "device.hpp"
#include "internal.hpp"

struct april_polys {
    uint64_t n = 0, nv = 0;
    int device = -1;
    void *mem = nullptr;            // one allocation: records, then vertices
    const int64_t *rec = nullptr;   // per polygon: vtx0, nv, xmin, ymin, xmax, ymax, x0, y0
    const int64_t *xy = nullptr;    // vertices, (x, y) interleaved
    uint64_t most = 0;              // vertices of the polygon with most
    int64_t lo[2] = {0, 0}, hi[2] = {0, 0};   // MBR of all
    int64_t *box = nullptr;         // boxes of 64 consecutive edges (xmin, ymin, xmax, ymax), see box_at
};

namespace april {
namespace {

constexpr int kRecWords = 8;

struct PolyView {
    const int64_t *rec, *xy, *box;
    uint64_t n;
};

// Edge boxes.  A polygon of more than 64 edges has a box for every 64
// consecutive ones.  Polygon k with first vertex v keeps its boxes from
// number v / 64 + k on: it has at most n / 64 + 1 of them, so the next
// polygon's begin behind them and no table of offsets is needed.
__device__ __forceinline__ uint64_t box_at(uint64_t v0, uint64_t k) { return (v0 >> 6) + k; }

struct RefineArgs {
    PolyView R, S;
    const uint32_t *r, *s;
    const uint8_t *verdict;
    uint8_t *out;
    unsigned long long *counts;
    unsigned int *xhead;
    uint32_t *left;      // pairs left to the second pass
    uint64_t n_pairs;
    uint32_t xcds;
    uint32_t grab;   // pairs per grab, 4 .. 64
    uint32_t grab_rest;   // of the second pass, 1 .. 64
};

typedef int64_t i64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ i64x2 gl128(const int64_t *p, uint64_t i) {
    return ((const i64x2 __attribute__((address_space(1))) *)p)[i];
}

__device__ __forceinline__ int sgn(__int128 v) { return (v > 0) - (v < 0); }

// sign of (b - a) x (c - a), 128-bit
__device__ __forceinline__ int orient(int64_t ax, int64_t ay, int64_t bx, int64_t by, int64_t cx, int64_t cy) {
    return sgn(__int128(bx - ax) * (cy - ay) - __int128(by - ay) * (cx - ax));
}

__device__ __forceinline__ bool within(int64_t a, int64_t b, int64_t p) { return min(a, b) <= p && p <= max(a, b); }

// do the closed segments ab and cd share a point?
__device__ __forceinline__ bool segments_meet(int64_t ax, int64_t ay, int64_t bx, int64_t by, int64_t cx, int64_t cy,
                                              int64_t dx, int64_t dy) {
    const int o1 = orient(ax, ay, bx, by, cx, cy), o2 = orient(ax, ay, bx, by, dx, dy);
    const int o3 = orient(cx, cy, dx, dy, ax, ay), o4 = orient(cx, cy, dx, dy, bx, by);
    if (o1 * o2 < 0 && o3 * o4 < 0) return true;    // proper crossing
    // an endpoint on the other segment (covers touching and collinear overlap)
    return (o1 == 0 && within(ax, bx, cx) && within(ay, by, cy)) ||
           (o2 == 0 && within(ax, bx, dx) && within(ay, by, dy)) ||
           (o3 == 0 && within(cx, dx, ax) && within(cy, dy, ay)) ||
           (o4 == 0 && within(cx, dx, bx) && within(cy, dy, by));
}

// The same predicates on coordinates relative to a pair's origin, every
// coordinate in [0, 2^31): differences fit in 32 bits, cross products in 64.
__device__ __forceinline__ int orient32(int32_t ax, int32_t ay, int32_t bx, int32_t by, int32_t cx, int32_t cy) {
    const int64_t v = int64_t(bx - ax) * int64_t(cy - ay) - int64_t(by - ay) * int64_t(cx - ax);
    return (v > 0) - (v < 0);
}

__device__ __forceinline__ bool within32(int32_t a, int32_t b, int32_t p) { return min(a, b) <= p && p <= max(a, b); }

// edges as (x0, y0, x1, y1)
__device__ __forceinline__ bool segments_meet32(int4 u, int4 w) {
    const int o1 = orient32(u.x, u.y, u.z, u.w, w.x, w.y), o2 = orient32(u.x, u.y, u.z, u.w, w.z, w.w);
    const int o3 = orient32(w.x, w.y, w.z, w.w, u.x, u.y), o4 = orient32(w.x, w.y, w.z, w.w, u.z, u.w);
    if (o1 * o2 < 0 && o3 * o4 < 0) return true;
    return (o1 == 0 && within32(u.x, u.z, w.x) && within32(u.y, u.w, w.y)) ||
           (o2 == 0 && within32(u.x, u.z, w.z) && within32(u.y, u.w, w.w)) ||
           (o3 == 0 && within32(w.x, w.z, u.x) && within32(w.y, w.w, u.y)) ||
           (o4 == 0 && within32(w.x, w.z, u.z) && within32(w.y, w.w, u.w));
}

__device__ __forceinline__ bool boxes_meet32(int4 u, int4 w) {
    return max(u.x, u.z) >= min(w.x, w.z) && min(u.x, u.z) <= max(w.x, w.z) && max(u.y, u.w) >= min(w.y, w.w) &&
           min(u.y, u.w) <= max(w.y, w.w);
}

// Does the edge u cross the horizontal line through (px, py) to the right of
// the point?  It crosses the line when exactly one endpoint lies strictly
// above; the crossing is right of the point when the point lies left of the
// upward-directed edge.  Never asked for a point on the edge.
__device__ __forceinline__ bool crosses_right32(int4 u, int32_t px, int32_t py) {
    if ((u.y > py) == (u.w > py)) return false;
    const int o = orient32(u.x, u.y, u.z, u.w, px, py);
    return u.w > u.y ? o > 0 : o < 0;
}

// A pair in relative coordinates (origin: lower-left corner of the MBRs'
// union); B = intersection of the MBRs.
struct Pair {
    uint64_t r0, s0;               // first vertex of each polygon
    uint32_t nr, ns;               // vertex (= edge) counts
    int64_t ox, oy;
    int32_t bx0, by0, bx1, by1;    // B
    int32_t rx, ry, sx, sy;        // first vertex of R and of S
    bool r_in_bs, s_in_br;         // R's first vertex in S's MBR, and S's in R's
};

enum : uint32_t { kDisjoint = 0, kNarrow = 1, kWide = 2 };

// Pairs of more edge pairs (of one polygon's with the other's), or with a
// polygon of more edges, go through the boxes.  7,200 pairs take about 0.1 ms
// there, whatever their size; through the chunks they take 0.17 ms at 250 x
// 250 edges, 0.36 ms at 400 x 400 and 0.17 ms at 1000 x 35, but 0.08 ms (the
// boxes 0.09) at 400 x 35.
constexpr uint64_t kManyEdgePairs = 1ull << 16;
constexpr uint32_t kManyEdges = 768;

// counter of the pairs that the first pass leaves to the second, and how many
// of them its list holds (in the scratch, behind the counters)
constexpr uint32_t kLeftCtr = kMaxCtrs - 1;
constexpr uint32_t kLeftCap = 1u << 16;

// workgroups of k_refine per CU: the residency its registers allow
constexpr int kRefineBlocksPerCU = 5, kRestBlocksPerCU = 4;

// mark pairs left for the second pass: wide ones, and those of many edges
constexpr uint8_t kWidePending = 0xFE, kManyPending = 0xFD;

__device__ __forceinline__ int4 rel_edge(const int64_t *xy, uint64_t p0, uint32_t e, uint32_t n, int64_t ox,
                                         int64_t oy) {
    const uint32_t e2 = e + 1 == n ? 0 : e + 1;
    const i64x2 a = gl128(xy, p0 + e), b = gl128(xy, p0 + e2);
    return make_int4(int32_t(a.x - ox), int32_t(a.y - oy), int32_t(b.x - ox), int32_t(b.y - oy));
}

__device__ __forceinline__ bool in_b(const Pair &q, int4 E) {
    return max(E.x, E.z) >= q.bx0 && min(E.x, E.z) <= q.bx1 && max(E.y, E.w) >= q.by0 && min(E.y, E.w) <= q.by1;
}

// write the lanes' edges flagged in `keep` to out[base ...] in lane order
__device__ __forceinline__ uint32_t append(int4 *out, uint32_t base, bool keep, int4 E) {
    const uint64_t m = __ballot(keep);
    if (keep) out[base + __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0))] = E;
    return uint32_t(__popcll(m));
}

// edges of one side staged in LDS per wave
constexpr uint32_t kEdgeChunk = 128;

// Append to `out` (from 0) the edges of a polygon (vertices [p0, p0 + n))
// that meet B, starting at edge *pos and taking whole blocks of 64 edges
// while at most kEdgeChunk can result; *pos becomes the first edge not
// scanned.  *cross accumulates, over every scanned edge, the crossings of
// the ray from (px, py).  Returns the count.  Whole wave.
__device__ uint32_t gather_edges(const int64_t *xy, uint64_t p0, uint32_t n, uint32_t &pos, const Pair &q,
                                 int32_t px, int32_t py, uint32_t &cross, int4 *out, uint32_t lane) {
    uint32_t cnt = 0;
    wave_lds_sync();   // earlier readers of `out` are done
    while (pos < n && cnt + 64 <= kEdgeChunk) {
        const uint32_t e = pos + lane;
        const bool v = e < n;
        const int4 E = rel_edge(xy, p0, v ? e : 0, n, q.ox, q.oy);
        cross += uint32_t(__popcll(__ballot(v && crosses_right32(E, px, py))));
        cnt += append(out, cnt, v && in_b(q, E), E);
        pos += 64;
    }
    wave_lds_sync();
    return cnt;
}

// Does any of the na edges in ea meet any of the nb edges in eb?  The
// na * nb pairs are dealt out 64 at a time (lane t takes pair t, row-major).
__device__ bool edges_meet(const int4 *ea, uint32_t na, const int4 *eb, uint32_t nb, uint32_t lane) {
    if (na == 0 || nb == 0) return false;
    const uint32_t total = na * nb, q = 64 / nb, rem = 64 % nb;
    uint32_t i = lane / nb, j = lane % nb;
    for (uint32_t t0 = 0; t0 < total; t0 += 64) {
        bool h = false;
        if (t0 + lane < total) {
            const int4 u = ea[i], w = eb[j];
            h = boxes_meet32(u, w) && segments_meet32(u, w);
        }
        if (__any(h)) return true;
        i += q;
        j += rem;
        if (j >= nb) {
            j -= nb;
            i++;
        }
    }
    return false;
}

// the containment decision once no boundary contact was found: cross_s
// counts the ray from R's first vertex over S's edges, cross_r the ray from
// S's first vertex over R's edges
__device__ __forceinline__ uint8_t contained(const Pair &q, uint32_t cross_s, uint32_t cross_r) {
    return ((q.r_in_bs && (cross_s & 1u)) || (q.s_in_br && (cross_r & 1u))) ? 1 : 0;
}

// Both polygons with at most 64 edges: one load round for both.
__device__ uint8_t refine_small(const RefineArgs &a, const Pair &q, int4 *ea, int4 *eb, uint32_t lane) {
    const bool vr = lane < q.nr, vs = lane < q.ns;
    const int4 Er = rel_edge(a.R.xy, q.r0, vr ? lane : 0, q.nr, q.ox, q.oy);
    const int4 Es = rel_edge(a.S.xy, q.s0, vs ? lane : 0, q.ns, q.ox, q.oy);
    wave_lds_sync();
    const uint32_t cr = append(ea, 0, vr && in_b(q, Er), Er);
    const uint32_t cs = append(eb, 0, vs && in_b(q, Es), Es);
    const uint32_t cross_s = uint32_t(__popcll(__ballot(vs && crosses_right32(Es, q.rx, q.ry))));
    const uint32_t cross_r = uint32_t(__popcll(__ballot(vr && crosses_right32(Er, q.sx, q.sy))));
    wave_lds_sync();
    if (edges_meet(ea, cr, eb, cs, lane)) return 1;
    return contained(q, cross_s, cross_r);
}

__device__ uint8_t refine_chunked(const RefineArgs &a, const Pair &q, int4 *ea, int4 *eb, uint32_t lane) {
    // chunks of R's edges against chunks of S's edges; S is gathered once
    // when its kept edges fit one chunk
    uint32_t pr = 0, cs = 0, cross_r = 0, cross_s = 0;
    bool s_counted = false, s_once = false;
    while (pr < q.nr) {
        const uint32_t cr = gather_edges(a.R.xy, q.r0, q.nr, pr, q, q.sx, q.sy, cross_r, ea, lane);
        if (cr == 0) continue;
        if (s_once) {
            if (edges_meet(ea, cr, eb, cs, lane)) return 1;
            continue;
        }
        uint32_t ps = 0, gathers = 0, cross = 0;
        do {
            cs = gather_edges(a.S.xy, q.s0, q.ns, ps, q, q.rx, q.ry, cross, eb, lane);
            gathers++;
            if (edges_meet(ea, cr, eb, cs, lane)) return 1;
        } while (ps < q.ns);
        if (!s_counted) {
            cross_s = cross;
            s_counted = true;
        }
        s_once = gathers == 1;
    }
    if (!s_counted && q.r_in_bs) {   // no kept edge of R: one pass over S for the ray count
        for (uint32_t e0 = 0; e0 < q.ns; e0 += 64) {
            const uint32_t e = e0 + lane;
            const bool v = e < q.ns;
            const int4 E = rel_edge(a.S.xy, q.s0, v ? e : 0, q.ns, q.ox, q.oy);
            cross_s += uint32_t(__popcll(__ballot(v && crosses_right32(E, q.rx, q.ry))));
        }
    }
    return contained(q, cross_s, cross_r);
}

// ------------------------------------------------------- many edges
//
// Two polygons of thousands of edges have few edges near each other, but
// testing the edges that meet B all-pairs is quadratic in them: 300 x 300
// polygons of 1k-20k vertices, 7,020 pairs, took 294 ms (its slowest pairs
// most of it; now 0.12 ms).  Edges that follow each other lie close together, so the boxes
// of 64 of them stand for them first: the wave holds 64 of R's boxes, one per
// lane, and goes over S's 64 at a time; only box pairs that meet have their
// 64 + 64 edges read, culled to the two boxes' intersection (which holds
// every point that they share) and tested.  The box tests are bounded by the
// latency of the loads, so that a lane's box is also tested against the union
// of R's 64 first, which drops most of S's at once.

struct EdgeSide {
    const int64_t *xy, *box;
    uint64_t v0;
    uint32_t n, boxes;
};

// box c, relative to the pair's origin, as (x0, y0, x1, y1); a polygon of at
// most 64 edges has one, B itself
__device__ __forceinline__ int4 side_box(const EdgeSide &d, const Pair &q, uint32_t c) {
    if (d.n <= 64) return make_int4(q.bx0, q.by0, q.bx1, q.by1);
    const i64x2 a = gl128(d.box, 2 * uint64_t(c)), b = gl128(d.box, 2 * uint64_t(c) + 1);
    return make_int4(int32_t(a.x - q.ox), int32_t(a.y - q.oy), int32_t(b.x - q.ox), int32_t(b.y - q.oy));
}

__device__ __forceinline__ bool boxes_overlap(int4 u, int4 w) {
    return u.x <= w.z && w.x <= u.z && u.y <= w.w && w.y <= u.w;
}

__device__ __forceinline__ int4 lane_box(int4 v, uint32_t k) {
    return make_int4(__builtin_amdgcn_readlane(v.x, k), __builtin_amdgcn_readlane(v.y, k),
                     __builtin_amdgcn_readlane(v.z, k), __builtin_amdgcn_readlane(v.w, k));
}

// the lane's edge of box c (an edge twice where there are fewer than 64)
__device__ __forceinline__ int4 side_edge(const EdgeSide &d, const Pair &q, uint32_t c, uint32_t lane) {
    return rel_edge(d.xy, d.v0, min(c * 64 + lane, d.n - 1), d.n, q.ox, q.oy);
}

__device__ __forceinline__ bool edge_in(int4 E, int4 b) {
    return max(E.x, E.z) >= b.x && min(E.x, E.z) <= b.z && max(E.y, E.w) >= b.y && min(E.y, E.w) <= b.w;
}

// crossings of the ray from (px, py) to the right: only edges in boxes that
// span the ray's height and reach beyond the point
__device__ uint32_t ray_crossings(const EdgeSide &d, const Pair &q, int32_t px, int32_t py, uint32_t lane) {
    uint32_t cross = 0;
    for (uint32_t c0 = 0; c0 < d.boxes; c0 += 64) {
        bool need = c0 + lane < d.boxes;
        if (need && d.n > 64) {
            const int4 b = side_box(d, q, c0 + lane);
            need = b.y <= py && b.w > py && b.z >= px;
        }
        uint64_t todo = __ballot(need);
        while (todo) {
            const uint32_t c = c0 + uint32_t(__builtin_ctzll(todo));
            todo &= todo - 1;
            const int4 E = side_edge(d, q, c, lane);
            cross += uint32_t(__popcll(__ballot(c * 64 + lane < d.n && crosses_right32(E, px, py))));
        }
    }
    return cross;
}

__device__ uint8_t refine_boxes(const EdgeSide &R, const EdgeSide &S, const Pair &q, int4 *ea, int4 *eb,
                                uint32_t lane) {
    const int4 B = make_int4(q.bx0, q.by0, q.bx1, q.by1);
    for (uint32_t g = 0; g < R.boxes; g += 64) {
        int4 rb = make_int4(INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN);   // meets nothing
        if (g + lane < R.boxes) {
            const int4 b = side_box(R, q, g + lane);
            if (boxes_overlap(b, B)) rb = b;
        }
        if (!__any(rb.x <= rb.z)) continue;
        int4 U = rb;
        for (int off = 32; off > 0; off >>= 1) {
            U.x = min(U.x, __shfl_xor(U.x, off));
            U.y = min(U.y, __shfl_xor(U.y, off));
            U.z = max(U.z, __shfl_xor(U.z, off));
            U.w = max(U.w, __shfl_xor(U.w, off));
        }
        for (uint32_t h = 0; h < S.boxes; h += 64) {
            const bool vs = h + lane < S.boxes;
            const int4 sb = side_box(S, q, vs ? h + lane : 0);
            uint64_t todo_s = __ballot(vs && boxes_overlap(sb, U) && boxes_overlap(sb, B));
            while (todo_s) {
                const uint32_t cs = uint32_t(__builtin_ctzll(todo_s));
                todo_s &= todo_s - 1;
                const int4 sbox = lane_box(sb, cs);
                uint64_t todo_r = __ballot(boxes_overlap(rb, sbox));
                if (!todo_r) continue;
                const int4 Es = side_edge(S, q, h + cs, lane);
                while (todo_r) {
                    const uint32_t cr = uint32_t(__builtin_ctzll(todo_r));
                    todo_r &= todo_r - 1;
                    const int4 rbox = lane_box(rb, cr);
                    const int4 Er = side_edge(R, q, g + cr, lane);
                    const int4 both = make_int4(max(rbox.x, sbox.x), max(rbox.y, sbox.y), min(rbox.z, sbox.z),
                                                min(rbox.w, sbox.w));
                    wave_lds_sync();
                    const uint32_t kr = append(ea, 0, (g + cr) * 64 + lane < R.n && edge_in(Er, both), Er);
                    const uint32_t ks = append(eb, 0, (h + cs) * 64 + lane < S.n && edge_in(Es, both), Es);
                    wave_lds_sync();
                    if (edges_meet(ea, kr, eb, ks, lane)) return 1;
                }
            }
        }
    }
    const uint32_t cross_s = q.r_in_bs ? ray_crossings(S, q, q.rx, q.ry, lane) : 0;
    const uint32_t cross_r = q.s_in_br ? ray_crossings(R, q, q.sx, q.sy, lane) : 0;
    return contained(q, cross_s, cross_r);
}

// --------------------------------------------------------- wide pairs

__device__ __forceinline__ bool in_box(const int64_t *rec, int64_t x, int64_t y) {
    return rec[2] <= x && x <= rec[4] && rec[3] <= y && y <= rec[5];
}

// one edge of A (uniform) against 64 edges of B per step, both culled to B
__device__ bool boundaries_meet_wide(const int64_t *axy, uint64_t a0, uint32_t na, const int64_t *bxy, uint64_t b0,
                                     uint32_t nb, int64_t bx0, int64_t by0, int64_t bx1, int64_t by1,
                                     uint32_t lane) {
    for (uint32_t q0 = 0; q0 < nb; q0 += 64) {
        const uint32_t q = q0 + lane;
        const bool qv = q < nb;
        const uint32_t qq = qv ? q : 0, q2 = qq + 1 == nb ? 0 : qq + 1;
        const i64x2 c = gl128(bxy, b0 + qq), d = gl128(bxy, b0 + q2);
        const bool qin =
            qv && max(c.x, d.x) >= bx0 && min(c.x, d.x) <= bx1 && max(c.y, d.y) >= by0 && min(c.y, d.y) <= by1;
        if (!__any(qin)) continue;
        i64x2 u = gl128(axy, a0);
        for (uint32_t k = 0; k < na; k++) {
            const uint32_t k2 = k + 1 == na ? 0 : k + 1;
            const i64x2 w = gl128(axy, a0 + k2);
            if (max(u.x, w.x) >= bx0 && min(u.x, w.x) <= bx1 && max(u.y, w.y) >= by0 && min(u.y, w.y) <= by1) {
                const bool h = qin && max(u.x, w.x) >= min(c.x, d.x) && min(u.x, w.x) <= max(c.x, d.x) &&
                               max(u.y, w.y) >= min(c.y, d.y) && min(u.y, w.y) <= max(c.y, d.y) &&
                               segments_meet(u.x, u.y, w.x, w.y, c.x, c.y, d.x, d.y);
                if (__any(h)) return true;
            }
            u = w;
        }
    }
    return false;
}

__device__ bool inside_wide(const int64_t *xy, uint64_t p0, uint32_t n, int64_t px, int64_t py, uint32_t lane) {
    uint32_t crossings = 0;
    for (uint32_t q0 = 0; q0 < n; q0 += 64) {
        const uint32_t q = q0 + lane;
        bool c = false;
        if (q < n) {
            const uint32_t q2 = q + 1 == n ? 0 : q + 1;
            const i64x2 u = gl128(xy, p0 + q), w = gl128(xy, p0 + q2);
            if ((u.y > py) != (w.y > py)) {
                const int o = orient(u.x, u.y, w.x, w.y, px, py);
                c = w.y > u.y ? o > 0 : o < 0;
            }
        }
        crossings += uint32_t(__popcll(__ballot(c)));
    }
    return crossings & 1u;
}

__device__ uint8_t refine_pair_wide(const RefineArgs &a, uint32_t r, uint32_t s, uint32_t lane) {
    const int64_t *br = a.R.rec + kRecWords * uint64_t(r), *bs = a.S.rec + kRecWords * uint64_t(s);
    const uint64_t r0 = uint64_t(br[0]), s0 = uint64_t(bs[0]);
    const uint32_t nr = uint32_t(br[1]), ns = uint32_t(bs[1]);
    const int64_t bx0 = max(br[2], bs[2]), by0 = max(br[3], bs[3]);
    const int64_t bx1 = min(br[4], bs[4]), by1 = min(br[5], bs[5]);
    if (boundaries_meet_wide(a.R.xy, r0, nr, a.S.xy, s0, ns, bx0, by0, bx1, by1, lane)) return 1;
    if (in_box(bs, br[6], br[7]) && inside_wide(a.S.xy, s0, ns, br[6], br[7], lane)) return 1;
    return in_box(br, bs[6], bs[7]) && inside_wide(a.R.xy, r0, nr, bs[6], bs[7], lane) ? 1 : 0;
}

// One wave per box number: find its polygon, reduce the box over the edges.
__global__ __launch_bounds__(256) void k_edge_boxes(const int64_t *rec, const int64_t *xy, uint64_t n,
                                                    uint64_t n_boxes, int64_t *box) {
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t waves = uint64_t(gridDim.x) * (blockDim.x / 64);
    for (uint64_t b = uint64_t(blockIdx.x) * (blockDim.x / 64) + (threadIdx.x >> 6); b < n_boxes; b += waves) {
        uint64_t lo = 0, hi = n;   // the last polygon whose boxes start at or before b
        while (hi - lo > 1) {
            const uint64_t mid = (lo + hi) / 2;
            if (box_at(uint64_t(rec[kRecWords * mid]), mid) <= b) lo = mid;
            else hi = mid;
        }
        const uint64_t v0 = uint64_t(rec[kRecWords * lo]), nv = uint64_t(rec[kRecWords * lo + 1]);
        const uint64_t e = (b - box_at(v0, lo)) * 64 + lane;
        if (nv <= 64 || e - lane >= nv) continue;
        int64_t x0 = INT64_MAX, y0 = INT64_MAX, x1 = INT64_MIN, y1 = INT64_MIN;
        if (e < nv) {
            const i64x2 u = gl128(xy, v0 + e), w = gl128(xy, v0 + (e + 1 == nv ? 0 : e + 1));
            x0 = min(u.x, w.x);
            y0 = min(u.y, w.y);
            x1 = max(u.x, w.x);
            y1 = max(u.y, w.y);
        }
        for (int off = 32; off > 0; off >>= 1) {
            x0 = min(x0, (int64_t)__shfl_xor((long long)x0, off));
            y0 = min(y0, (int64_t)__shfl_xor((long long)y0, off));
            x1 = max(x1, (int64_t)__shfl_xor((long long)x1, off));
            y1 = max(y1, (int64_t)__shfl_xor((long long)y1, off));
        }
        if (lane < 4) box[4 * b + lane] = lane == 0 ? x0 : lane == 1 ? y0 : lane == 2 ? x1 : y1;
    }
}

// ------------------------------------------------------------- kernels

__device__ __forceinline__ uint32_t rl32(uint32_t v, uint32_t k) { return uniform(__builtin_amdgcn_readlane(v, k)); }
__device__ __forceinline__ int32_t rli(int32_t v, uint32_t k) { return int32_t(rl32(uint32_t(v), k)); }
__device__ __forceinline__ uint64_t rl64(uint64_t v, uint32_t k) {
    return uint64_t(rl32(uint32_t(v), k)) | (uint64_t(rl32(uint32_t(v >> 32), k)) << 32);
}

// First pass (REST false): every pair but those of polygons with many edges
// and wide ones, which it marks; second pass (REST): those.  Two kernels: with
// the box path in it the first needs more registers, and a 1.13M-pair call of
// small polygons took 632 us, not 590.
template <bool REST>
__global__ __launch_bounds__(kBlock) void k_refine(RefineArgs a) {
    __shared__ int4 lds[kWavesPerBlock][2][kEdgeChunk];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int4 *ea = lds[wave][0], *eb = lds[wave][1];
    unsigned long long c_hit = 0, c_tested = 0;
    // second pass: pair by pair from the list, or, with more pairs than it
    // holds, from the marks
    const uint32_t n_left = REST ? uniform(a.xhead[kLeftCtr * kCtrStride]) : 0;
    const bool listed = REST && n_left <= kLeftCap;
    uint32_t next = blockIdx.x * kWavesPerBlock + wave;
    if (listed && next >= n_left) return;
    const uint32_t my_xcd = blockIdx.x % a.xcds, G = REST ? a.grab_rest : a.grab;
    for (uint32_t k = 0; k < a.xcds; k++) {
        const uint32_t seg = (my_xcd + k) % a.xcds;
        const uint64_t lo = a.n_pairs * seg / a.xcds, hi = a.n_pairs * (seg + 1) / a.xcds;
        const uint32_t ctr = REST ? a.xcds + seg : seg;
        if (!listed && k > 0 && range_drained(a.xhead, ctr, lo, hi, lane)) continue;
        for (;;) {
            uint64_t g0;
            if (listed) {
                if (next >= n_left) break;
                g0 = uniform(a.left[next]);
                next += gridDim.x * kWavesPerBlock;
            } else {
                unsigned int got = 0;
                if (lane == 0) got = atomicAdd(&a.xhead[ctr * kCtrStride], G);
                g0 = lo + uniform(__shfl(got, 0));
                if (g0 >= hi) break;
            }
            const uint64_t p = g0 + lane;
            bool mine = listed ? lane == 0 : lane < G && p < hi;
            if (REST && mine) mine = a.out[p] == kWidePending || a.out[p] == kManyPending;
            if (REST && !__any(mine)) continue;
            uint32_t out = APRIL_BAD_PAIR, kind = kDisjoint;
            bool test = false;
            // this lane's pair: ids, verdict, both records
            Pair m = {};
            uint32_t r = 0, s = 0;
            if (mine) {
                r = a.r[p];
                s = a.s[p];
                if (REST) {
                    test = true;
                } else if (r < a.R.n && s < a.S.n) {
                    const uint8_t v = a.verdict ? a.verdict[p] : uint8_t(APRIL_INDECISIVE);
                    if (v == APRIL_TN) out = 0;
                    else if (v == APRIL_TH) out = 1;
                    else test = true;
                }
                if (test) {
                    const int64_t *pr = a.R.rec + kRecWords * uint64_t(r), *ps = a.S.rec + kRecWords * uint64_t(s);
                    const i64x2 r01 = gl128(pr, 0), r23 = gl128(pr, 1), r45 = gl128(pr, 2), r67 = gl128(pr, 3);
                    const i64x2 s01 = gl128(ps, 0), s23 = gl128(ps, 1), s45 = gl128(ps, 2), s67 = gl128(ps, 3);
                    const int64_t bx0 = max(r23.x, s23.x), by0 = max(r23.y, s23.y);
                    const int64_t bx1 = min(r45.x, s45.x), by1 = min(r45.y, s45.y);
                    const int64_t ux0 = min(r23.x, s23.x), uy0 = min(r23.y, s23.y);
                    const int64_t ux1 = max(r45.x, s45.x), uy1 = max(r45.y, s45.y);
                    if (bx0 > bx1 || by0 > by1) {
                        kind = kDisjoint;   // the MBRs do not meet
                    } else if (uint64_t(ux1) - uint64_t(ux0) >= (1ull << 31) ||
                               uint64_t(uy1) - uint64_t(uy0) >= (1ull << 31)) {
                        kind = kWide;       // (unsigned differences: exact for any int64)
                    } else {
                        kind = kNarrow;
                        m.r0 = uint64_t(r01.x);
                        m.nr = uint32_t(r01.y);
                        m.s0 = uint64_t(s01.x);
                        m.ns = uint32_t(s01.y);
                        m.ox = ux0;
                        m.oy = uy0;
                        m.bx0 = int32_t(bx0 - ux0);
                        m.by0 = int32_t(by0 - uy0);
                        m.bx1 = int32_t(bx1 - ux0);
                        m.by1 = int32_t(by1 - uy0);
                        m.rx = int32_t(r67.x - ux0);
                        m.ry = int32_t(r67.y - uy0);
                        m.sx = int32_t(s67.x - ux0);
                        m.sy = int32_t(s67.y - uy0);
                        m.r_in_bs = s23.x <= r67.x && r67.x <= s45.x && s23.y <= r67.y && r67.y <= s45.y;
                        m.s_in_br = r23.x <= s67.x && s67.x <= r45.x && r23.y <= s67.y && s67.y <= r45.y;
                    }
                }
            }
            const bool many = uint64_t(m.nr) * m.ns > kManyEdgePairs || max(m.nr, m.ns) > kManyEdges;
            uint64_t todo = __ballot(REST ? test : test && kind == kNarrow && !many);
            if (!REST && test && kind != kNarrow) out = kind == kWide ? kWidePending : 0;
            if (!REST && test && kind == kNarrow && many) out = kManyPending;
            if (!REST) {
                const bool mark = out == kWidePending || out == kManyPending;
                const uint64_t left = __ballot(mark);
                if (left) {
                    unsigned int at = 0;
                    if (lane == 0) at = atomicAdd(&a.xhead[kLeftCtr * kCtrStride], uint32_t(__popcll(left)));
                    const uint64_t slot = uint64_t(__shfl(at, 0)) + uint32_t(__popcll(left & ((1ull << lane) - 1)));
                    if (mark && slot < kLeftCap) a.left[slot] = uint32_t(p);
                }
            }
            while (todo) {
                const uint32_t k2 = uint32_t(__builtin_ctzll(todo));
                todo &= todo - 1;
                if (REST && rl32(kind, k2) == kWide) {
                    const uint32_t vw = refine_pair_wide(a, rl32(r, k2), rl32(s, k2), lane);
                    out = lane == k2 ? vw : out;
                    continue;
                }
                Pair q;
                q.r0 = rl64(m.r0, k2);
                q.s0 = rl64(m.s0, k2);
                q.nr = rl32(m.nr, k2);
                q.ns = rl32(m.ns, k2);
                q.ox = int64_t(rl64(uint64_t(m.ox), k2));
                q.oy = int64_t(rl64(uint64_t(m.oy), k2));
                q.bx0 = rli(m.bx0, k2);
                q.by0 = rli(m.by0, k2);
                q.bx1 = rli(m.bx1, k2);
                q.by1 = rli(m.by1, k2);
                q.rx = rli(m.rx, k2);
                q.ry = rli(m.ry, k2);
                q.sx = rli(m.sx, k2);
                q.sy = rli(m.sy, k2);
                q.r_in_bs = rl32(m.r_in_bs, k2) != 0;
                q.s_in_br = rl32(m.s_in_br, k2) != 0;
                uint32_t v;
                if (!REST) {
                    v = q.nr <= 64 && q.ns <= 64 ? refine_small(a, q, ea, eb, lane)
                                                 : refine_chunked(a, q, ea, eb, lane);
                } else {
                    const EdgeSide er{a.R.xy, a.R.box + 4 * box_at(q.r0, rl32(r, k2)), q.r0, q.nr, (q.nr + 63) / 64};
                    const EdgeSide es{a.S.xy, a.S.box + 4 * box_at(q.s0, rl32(s, k2)), q.s0, q.ns, (q.ns + 63) / 64};
                    v = refine_boxes(er, es, q, ea, eb, lane);
                }
                out = lane == k2 ? v : out;
            }
            if (mine) {
                a.out[p] = uint8_t(out);
                c_hit += out == 1;
                c_tested += !REST && test;
            }
        }
    }
    if (a.counts) {
        for (int off = 32; off > 0; off >>= 1) {
            c_hit += __shfl_down(c_hit, off);
            c_tested += __shfl_down(c_tested, off);
        }
        const unsigned long long v[2] = {c_hit, c_tested};
        if (lane == 0) add_totals(a.xhead, blockIdx.x * kWavesPerBlock + wave, v, 2);
    }
}

// do the two collections together span 2^31 lattice units or more in x
// (axis 0) or y?
bool wider(const april_polys_t *R, const april_polys_t *S, int axis) {
    const int64_t lo = std::min(R->lo[axis], S->lo[axis]), hi = std::max(R->hi[axis], S->hi[axis]);
    return uint64_t(hi) - uint64_t(lo) >= (1ull << 31);
}

PolyView view(const april_polys_t *P) { return PolyView{P->rec, P->xy, P->box, P->n}; }

}  // namespace
}  // namespace april

using namespace april;

extern "C" int april_polys_to_device(const double *xy, const uint64_t *vtx_off, uint64_t n, uint32_t flags,
                                     void *hip_stream, april_polys_t **out) {
    clear_error();
    if (!xy || !vtx_off || !out) return fail(APRIL_E_INVALID, "NULL argument");
    if (n == 0) return fail(APRIL_E_INVALID, "no polygons");
    if (flags & ~APRIL_STRICT) return fail(APRIL_E_INVALID, "unknown flags");
    const bool strict = flags & APRIL_STRICT;
    const uint64_t nv = vtx_off[n];
    for (uint64_t k = 0; k < n; k++)
        if (vtx_off[k + 1] < vtx_off[k] + 3 || vtx_off[k + 1] - vtx_off[k] > (1ull << 31))
            return fail(APRIL_E_INVALID, "polygon with < 3 or > 2^31 vertices");
    // host staging: records [8n], then vertices [2nv] (one block, one copy)
    const uint64_t words = uint64_t(kRecWords) * n + 2 * (nv - vtx_off[0]);
    std::vector<int64_t> h;
    try {
        h.resize(words);
    } catch (...) {
        return fail(APRIL_E_NOMEM, "out of host memory");
    }
    int64_t *rec = h.data(), *vxy = rec + uint64_t(kRecWords) * n;
    std::atomic<int> err{0};
    const int T = int(std::min<uint64_t>(host_threads(), n));
    parallel(T, [&](int t) {
        for (uint64_t k = n * uint64_t(t) / uint64_t(T); k < n * uint64_t(t + 1) / uint64_t(T); k++) {
            int64_t b[4] = {INT64_MAX, INT64_MAX, INT64_MIN, INT64_MIN};
            for (uint64_t v = vtx_off[k]; v < vtx_off[k + 1]; v++) {
                int64_t c[2];
                for (int d = 0; d < 2; d++) {
                    const double q = xy[2 * v + d] * 1073741824.0;
                    const double rr = std::nearbyint(q);
                    if (!(std::fabs(rr) < 4.6e18)) { err.store(APRIL_E_INVALID); return; }
                    if (strict && rr != q) { err.store(APRIL_E_INVALID); return; }
                    c[d] = int64_t(rr);
                }
                const uint64_t i = v - vtx_off[0];
                vxy[2 * i] = c[0];
                vxy[2 * i + 1] = c[1];
                b[0] = std::min(b[0], c[0]);
                b[1] = std::min(b[1], c[1]);
                b[2] = std::max(b[2], c[0]);
                b[3] = std::max(b[3], c[1]);
            }
            int64_t *o = rec + uint64_t(kRecWords) * k;
            const uint64_t first = vtx_off[k] - vtx_off[0];
            o[0] = int64_t(first);
            o[1] = int64_t(vtx_off[k + 1] - vtx_off[k]);
            for (int d = 0; d < 4; d++) o[2 + d] = b[d];
            o[6] = vxy[2 * first];
            o[7] = vxy[2 * first + 1];
        }
    });
    if (err.load()) return fail(APRIL_E_INVALID, "non-lattice coordinate (APRIL_STRICT) or coordinate out of range");
    auto *P = new (std::nothrow) april_polys;
    if (!P) return fail(APRIL_E_NOMEM, "out of host memory");
    int dev = 0;
    const uint64_t n_boxes = ((nv - vtx_off[0]) >> 6) + n;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipMalloc(&P->mem, (words + 4 * n_boxes) * sizeof(int64_t)) != hipSuccess) {
        delete P;
        return fail(APRIL_E_NOMEM, "device allocation of the polygons failed");
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    int64_t *d = static_cast<int64_t *>(P->mem);
    P->rec = d;
    P->xy = d + uint64_t(kRecWords) * n;
    P->box = d + words;
    bool ok = hipMemcpyAsync(P->mem, h.data(), words * sizeof(int64_t), hipMemcpyHostToDevice, stream) == hipSuccess;
    if (ok) {
        k_edge_boxes<<<dim3(uint32_t(std::min<uint64_t>((n_boxes + 3) / 4, 8192))), dim3(256), 0, stream>>>(
            P->rec, P->xy, n, n_boxes, P->box);
        ok = hipGetLastError() == hipSuccess;
    }
    if (hipStreamSynchronize(stream) != hipSuccess || !ok) {   // the staging buffer dies here
        (void)hipFree(P->mem);
        delete P;
        return fail(APRIL_E_HIP, "copy of the polygons to the device failed");
    }
    for (uint64_t k = 0; k < n; k++) {
        const int64_t *o = rec + uint64_t(kRecWords) * k;
        P->most = std::max(P->most, uint64_t(o[1]));
        for (int c = 0; c < 2; c++) {
            P->lo[c] = k ? std::min(P->lo[c], o[2 + c]) : o[2 + c];
            P->hi[c] = k ? std::max(P->hi[c], o[4 + c]) : o[4 + c];
        }
    }
    P->n = n;
    P->nv = nv - vtx_off[0];
    P->device = dev;
    *out = P;
    return APRIL_OK;
}

extern "C" void april_polys_free(april_polys_t *P) {
    if (!P) return;
    if (P->mem) (void)hipFree(P->mem);
    delete P;
}

extern "C" int april_refine_pairs(const april_polys_t *R, const april_polys_t *S, const uint32_t *d_r,
                                  const uint32_t *d_s, uint64_t n_pairs, const uint8_t *d_verdict, uint8_t *d_out,
                                  unsigned long long *d_counts, void *hip_stream) {
    clear_error();
    if (!R || !S) return fail(APRIL_E_INVALID, "NULL polygon collection");
    if (n_pairs && (!d_r || !d_s || !d_out)) return fail(APRIL_E_INVALID, "NULL pair or output array");
    if (n_pairs >= (1ull << 32)) return fail(APRIL_E_INVALID, "more than 2^32 - 1 pairs in one call");
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    int dev = 0;
    APRIL_HIP_TRY(hipGetDevice(&dev));
    if (R->device != dev || S->device != dev) return fail(APRIL_E_INVALID, "polygons live on another device");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    RefineArgs a;
    a.R = view(R);
    a.S = view(S);
    a.r = d_r;
    a.s = d_s;
    a.verdict = d_verdict;
    a.out = d_out;
    a.counts = d_counts;
    a.n_pairs = n_pairs;
    a.xcds = uint32_t(std::min(xcd_count(st->cus), int(kLeftCtr) / 2));   // two passes' counters
    // 64 pairs per grab, fewer when that would leave waves idle (about two
    // grabs per wave), but at least 4: each grab costs an atomic (1,650 pairs
    // of small polygons take 45 us with grabs of 1, 39 with 4).  The second
    // pass's pairs cost more than that, so it goes down to 1.
    const uint64_t blocks = uint64_t(st->cus) * kRefineBlocksPerCU, waves = blocks * kWavesPerBlock;
    a.grab_rest = uint32_t(std::min<uint64_t>(64, std::max<uint64_t>(1, n_pairs / (waves * 2))));
    a.grab = std::max(4u, a.grab_rest);
    // per-XCD range counters (and the second pass's list) in a stream-ordered
    // scratch, so calls on different streams never share them
    // (the second pass only where the collections can have pairs for it)
    const bool rest = R->most > kManyEdgePairs / S->most || std::max(R->most, S->most) > kManyEdges || wider(R, S, 0) || wider(R, S, 1);
    void *ws = nullptr;
    hipError_t e = hipMallocAsync(&ws, kCtrBytes + (rest ? 4ull * kLeftCap : 0), stream);
    if (e != hipSuccess) return fail(APRIL_E_NOMEM, std::string("refine scratch: ") + hipGetErrorString(e));
    a.xhead = static_cast<unsigned int *>(ws);
    a.left = reinterpret_cast<uint32_t *>(static_cast<char *>(ws) + kCtrBytes);
    k_zero_ctrs<<<1, 64, 0, stream>>>(a.xhead);
    e = hipGetLastError();
    if (e == hipSuccess && n_pairs) {
        k_refine<false><<<dim3(uint32_t(blocks)), dim3(kBlock), 0, stream>>>(a);
        e = hipGetLastError();
        if (e == hipSuccess && rest) {
            k_refine<true><<<dim3(uint32_t(st->cus * kRestBlocksPerCU)), dim3(kBlock), 0, stream>>>(a);
            e = hipGetLastError();
        }
    }
    if (e == hipSuccess && d_counts) {
        k_sum_totals<<<1, 64, 0, stream>>>(a.xhead, d_counts, 2);
        e = hipGetLastError();
    }
    APRIL_HIP_TRY(hipFreeAsync(ws, stream));
    if (e != hipSuccess) return fail(APRIL_E_HIP, std::string("refine launch: ") + hipGetErrorString(e));
    return APRIL_OK;
}
