// GPU construction of APRIL A- and F-lists (Sec. 6), for a whole collection
// at once.  The lists are identical to the host builder's (build.cpp): the
// same exact edge traversal, the same centre-line crossing rule, the same
// classes.  No cell is ever sorted: an aligned block of 64 x 64 cells is one
// contiguous range of Hilbert ids, so a polygon is rasterized block by block
// into bit arrays that are laid out in Hilbert order, where an interval is a
// run of ones.
//
//  1. one thread per vertex: lattice coordinates relative to the grid origin
//     (in place) and the checks (lattice, grid ring);
//  2. one wave per 64 consecutive edges: their box; one wave per polygon:
//     its extent in cells, which gives its blocks;
//  3. every block of every polygon (of those of many blocks, where it pays: every
//     one that is not empty) is an item with the key (polygon, Hilbert id of the block); a
//     radix sort of these keys is the lists' order;
//  4. one wave per item rasterizes it and counts the interval starts in it;
//     whether an interval runs on from the block before or into the next one
//     is a bit at either end, which a pass over the items settles;
//  5. scans give each item its place in the lists, and the items are
//     rasterized again and written there (storing them would take more
//     memory than the lists).
//
// An item, by one wave (k_items).  Edges that only pass left of the block
// change the parity of whole rows, which two comparisons per edge (or per 64
// edges: their first and last vertex tell) give as a 64-bit mask; edges to the
// right or above or below change nothing.  The rows of the edges that meet the
// block are dealt out to the lanes, one (edge, row) each, so that long and
// short edges fill the wave alike; a lane sets the cells whose closed square
// the edge meets in that row (T), those whose interior it crosses (C), and
// toggles the parity behind the crossing of the row's centre line.  Then lane
// l owns 64 cells in Hilbert order (8 x 8 of them): a cell that is not
// touched is inside when its centre is, and all of a run of such cells are
// alike, so one look at the parity per run and word decides (Alg. 3's gap
// test), and one per cell touched only on its border.
//
// Against emitting a 64-bit key per touched cell, sorting and compacting
// them, as this file did before: 50k polygons of the at-scale collection
// (715 cells and 327 intervals each) took 12.6 ms of kernels and 3.1 GB of
// scratch, whose mapping and unmapping took up to 80 ms more in a call; now they
// take 2.0 ms and 55 MB, and the whole call with a filter call behind it 5.0
// ms, not 20.7 to 98.  k_items takes 0.65 ms to count and 1.04 to write, at
// 0.87 to 0.89 of the VALU issue peak (783 instructions per item, 1,270 with the
// writing).  Blocks of 64 x 64 cells, because a wave then has one word of 64
// cells per lane and one row of cells per lane; at scale a polygon has nine,
// with 55 edge rows each, about one per lane.
//
// Host synchronizations read the sizes that the buffers need (one more where
// polygons have many blocks) and, at the end, the longest lists; the last one
// makes the lists complete for any stream.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <new>

#include "device.hpp"
#include "internal.hpp"

namespace april {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ int64_t fdiv(int64_t a, int64_t b) {   // floor(a / b), b > 0
    const int64_t q = a / b;
    return (a % b != 0 && a < 0) ? q - 1 : q;
}
__device__ __forceinline__ int64_t fdiv(__int128 a, __int128 b) {
    const __int128 q = a / b;
    return int64_t((a % b != 0 && a < 0) ? q - 1 : q);
}
template <typename T>
__device__ __forceinline__ int64_t cdiv(T a, T b) { return -fdiv(T(-a), b); }

// Hilbert curve, the library's variant: quadrants lower-left, upper-left,
// upper-right, lower-right; the first sub-curve transposed, the last one
// reflected in the anti-diagonal.  A state is one of the four symmetries
// (0 identity, 1 transpose, 2 anti-transpose, 3 half turn); they compose by
// XOR.
__device__ __forceinline__ void sym(uint32_t s, uint32_t bx, uint32_t by, uint32_t &ox, uint32_t &oy) {
    const uint32_t swap = (s ^ (s >> 1)) & 1u, flip = (s >> 1) & 1u;
    ox = (swap ? by : bx) ^ flip;
    oy = (swap ? bx : by) ^ flip;
}
__device__ __forceinline__ uint32_t child(uint32_t digit) { return digit == 0 ? 1u : digit == 3 ? 2u : 0u; }

__device__ uint32_t hilbert_d(int order, uint32_t x, uint32_t y) {
    uint32_t state = 0, d = 0;
    for (int lvl = order - 1; lvl >= 0; lvl--) {
        uint32_t qx, qy;
        sym(state, (x >> lvl) & 1u, (y >> lvl) & 1u, qx, qy);
        const uint32_t digit = (qx * 3u) ^ qy;   // (0,0)->0 (0,1)->1 (1,1)->2 (1,0)->3
        d = (d << 2) | digit;
        state ^= child(digit);
    }
    return d;
}

__device__ void hilbert_xy(int order, uint32_t d, uint32_t &x, uint32_t &y) {
    uint32_t state = 0, X = 0, Y = 0;
    for (int lvl = order - 1; lvl >= 0; lvl--) {
        const uint32_t digit = (d >> (2 * lvl)) & 3u;
        uint32_t bx, by;
        sym(state, digit >> 1, (digit ^ (digit >> 1)) & 1u, bx, by);   // quadrant of the digit
        X = (X << 1) | bx;
        Y = (Y << 1) | by;
        state ^= child(digit);
    }
    x = X;
    y = Y;
}

struct Geo {
    double x0, y0;     // grid origin
    int64_t w;         // cell side, lattice units
    double inv_w;      // 1 / w
    float inv_wf, inv_2wf;
    int64_t cells;     // 2^order
    int order;
    int border;        // order of the grid of blocks (0 when the grid is one block or less)
    uint32_t strict;
};

// error word: (polygon << 32) | (vertex in polygon << 8) | code; the
// smallest wins, so the report names the first failing polygon and, in it,
// the first failing check in vertex order (as the host builder does)
enum : uint64_t { kErrGrid = 1, kErrLattice = 2, kErrDistinct = 3 };
constexpr uint64_t kErrNoVertex = 0xffffff;

typedef int64_t i64x2 __attribute__((ext_vector_type(2)));

// xy: float64 coordinates in, int64 lattice coordinates out (in place)
__global__ void k_vertices(i64x2 *xy, const uint64_t *voff, uint64_t n, uint64_t nv, Geo g,
                           unsigned long long *err) {
    const uint64_t v = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    const i64x2 in = xy[v];
    uint64_t code = 0;
    int64_t c[2] = {0, 0};
    for (int a = 0; a < 2 && !code; a++) {
        const double q = (__longlong_as_double(a ? in.y : in.x) - (a ? g.y0 : g.x0)) * 1073741824.0;
        const double r = rint(q);
        if (!(fabs(r) < 4.0e15)) code = kErrGrid;
        else if (g.strict && r != q) code = kErrLattice;
        else c[a] = int64_t(r);
    }
    // the outer ring of cells must stay untouched
    if (!code && (c[0] <= g.w || c[1] <= g.w || c[0] >= (g.cells - 1) * g.w || c[1] >= (g.cells - 1) * g.w))
        code = kErrGrid;
    xy[v] = i64x2{c[0], c[1]};
    if (code) {
        uint64_t lo = 0, hi = n;   // polygon of vertex v: voff[lo] <= v < voff[hi]
        while (hi - lo > 1) {
            const uint64_t mid = (lo + hi) / 2;
            if (voff[mid] <= v) lo = mid;
            else hi = mid;
        }
        const uint64_t vl = min<uint64_t>(v - voff[lo], kErrNoVertex - 1);
        atomicMin(err, (unsigned long long)((lo << 32) | (vl << 8) | code));
    }
}

// Boxes of 64 consecutive edges: polygon k keeps its boxes from number
// voff[k] / 64 + k on (it has at most its vertices / 64 + 1 of them, so the
// next polygon's begin behind them).
struct EdgeBox {
    int64_t x0, y0, x1, y1;
};

__device__ __forceinline__ uint64_t box_at(uint64_t v0, uint64_t k) { return (v0 >> 6) + k; }

// the lane's edge of a polygon (vertices [v0, v0 + nv)): edge e from vertex e
__device__ __forceinline__ void load_edge(const i64x2 *xy, uint64_t v0, uint64_t nv, uint64_t e, i64x2 &a, i64x2 &b) {
    a = xy[v0 + e];
    b = xy[v0 + (e + 1 == nv ? 0 : e + 1)];
}

struct PolyArgs {
    const i64x2 *xy;
    const uint64_t *voff;
    uint64_t n, n_boxes;
    EdgeBox *box;
    uint32_t *distinct;        // per box: edges with two different ends
    unsigned long long *bound; // upper bound of the cells that all edges meet
    Geo g;
};

// The cells that an edge meets number at most its extent in x plus three per
// row (a row's first and last cell are shared with its neighbours' or touched
// at a corner only).
__global__ __launch_bounds__(256) void k_edge_boxes(PolyArgs a) {
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t waves = uint64_t(gridDim.x) * (blockDim.x / 64);
    unsigned long long cells = 0;
    for (uint64_t b = uint64_t(blockIdx.x) * (blockDim.x / 64) + (threadIdx.x >> 6); b < a.n_boxes; b += waves) {
        uint64_t lo = 0, hi = a.n;   // the last polygon whose boxes start at or before b
        while (hi - lo > 1) {
            const uint64_t mid = (lo + hi) / 2;
            if (box_at(a.voff[mid], mid) <= b) lo = mid;
            else hi = mid;
        }
        const uint64_t v0 = a.voff[lo], nv = a.voff[lo + 1] - v0;
        const uint64_t e = (b - box_at(v0, lo)) * 64 + lane;
        if (e - lane >= nv) continue;   // a number that no box has
        EdgeBox x{INT64_MAX, INT64_MAX, INT64_MIN, INT64_MIN};
        bool two = false;
        if (e < nv) {
            i64x2 u, v;
            load_edge(a.xy, v0, nv, e, u, v);
            x = EdgeBox{min(u.x, v.x), min(u.y, v.y), max(u.x, v.x), max(u.y, v.y)};
            two = u.x != v.x || u.y != v.y;
            cells += uint64_t(double(x.x1 - x.x0) * a.g.inv_w) + 3 * uint64_t(double(x.y1 - x.y0) * a.g.inv_w) + 16;
        }
        for (int off = 32; off > 0; off >>= 1) {
            x.x0 = min(x.x0, (int64_t)__shfl_xor((long long)x.x0, off));
            x.y0 = min(x.y0, (int64_t)__shfl_xor((long long)x.y0, off));
            x.x1 = max(x.x1, (int64_t)__shfl_xor((long long)x.x1, off));
            x.y1 = max(x.y1, (int64_t)__shfl_xor((long long)x.y1, off));
        }
        const uint32_t d = uint32_t(__popcll(__ballot(two)));
        if (lane == 0) {
            a.box[b] = x;
            a.distinct[b] = d;
        }
    }
    for (int off = 32; off > 0; off >>= 1) cells += __shfl_down(cells, off);
    // one addition per workgroup: 65,536 waves adding to one word took 0.5 ms
    __shared__ unsigned long long part[4];
    if (lane == 0) part[threadIdx.x >> 6] = cells;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(a.bound, part[0] + part[1] + part[2] + part[3]);
}

// A polygon's blocks: x0, y0 of the first, and how many in x and y.
struct Blocks {
    uint16_t x0, y0, nx, ny;
};

__device__ __forceinline__ int64_t floor_w(int64_t v, const Geo &g) {   // floor(v / w), v >= 0
    int64_t q = int64_t(double(v) * g.inv_w);
    const int64_t r = v - q * g.w;
    return r < 0 ? q - 1 : r >= g.w ? q + 1 : q;
}

// Polygons of this many blocks or more have an item only for the blocks that
// are not empty (k_block_rows): a sliver across the grid has 2^18 blocks and an
// edge in a thousand of them.  With fewer blocks, empty ones included, slivers
// take half of what they took when every cell had a key.
constexpr uint32_t kManyBlocks = 256;
// That takes two further passes over their edges and a synchronization, 40 to 50
// us, so it is done where such polygons have this many blocks together.  Without
// and with it: a sliver of 5k blocks 340 and 352 us, of 20k 389 and 369, of 80k
// 595 and 414; stars, of whose blocks a third are empty, 350 and 396 us at 2.5k
// blocks, 523 and 569 at 40k, 1,280 and 1,253 at 160k.
constexpr uint64_t kManyTotal = 1ull << 16;

// One wave per polygon; item count of polygon k in items[k] (items[n] = 0).
// Polygons of many blocks are listed, found[0] of them with found[1] blocks.
__global__ __launch_bounds__(256) void k_polygons(PolyArgs a, Blocks *blocks, uint64_t *items, uint32_t *many,
                                                  unsigned long long *found, unsigned long long *err) {
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t waves = uint64_t(gridDim.x) * (blockDim.x / 64);
    for (uint64_t k = uint64_t(blockIdx.x) * (blockDim.x / 64) + (threadIdx.x >> 6); k < a.n; k += waves) {
        const uint64_t v0 = a.voff[k], nv = a.voff[k + 1] - v0, b0 = box_at(v0, k), nb = (nv + 63) / 64;
        EdgeBox x{INT64_MAX, INT64_MAX, INT64_MIN, INT64_MIN};
        uint32_t d = 0;
        for (uint64_t b = lane; b < nb; b += 64) {
            const EdgeBox o = a.box[b0 + b];
            x = EdgeBox{min(x.x0, o.x0), min(x.y0, o.y0), max(x.x1, o.x1), max(x.y1, o.y1)};
            d = min(3u, d + a.distinct[b0 + b]);
        }
        for (int off = 32; off > 0; off >>= 1) {
            x.x0 = min(x.x0, (int64_t)__shfl_xor((long long)x.x0, off));
            x.y0 = min(x.y0, (int64_t)__shfl_xor((long long)x.y0, off));
            x.x1 = max(x.x1, (int64_t)__shfl_xor((long long)x.x1, off));
            x.y1 = max(x.y1, (int64_t)__shfl_xor((long long)x.y1, off));
            d = min(3u, d + __shfl_xor(d, off));
        }
        if (lane == 0) {
            if (d < 3) atomicMin(err, (unsigned long long)((k << 32) | (kErrNoVertex << 8) | kErrDistinct));
            // cells whose closed square the box meets; inside the grid's outer
            // ring unless a vertex was in error, when the call ends before the
            // blocks are used
            const int64_t top = a.g.cells - 1;
            const int64_t i0 = min(top, max<int64_t>(0, floor_w(x.x0 + a.g.w - 1, a.g) - 1));
            const int64_t j0 = min(top, max<int64_t>(0, floor_w(x.y0 + a.g.w - 1, a.g) - 1));
            const int64_t i1 = max(i0, min(top, floor_w(x.x1, a.g))), j1 = max(j0, min(top, floor_w(x.y1, a.g)));
            Blocks c;
            c.x0 = uint16_t(i0 >> 6);
            c.y0 = uint16_t(j0 >> 6);
            c.nx = uint16_t((i1 >> 6) - (i0 >> 6) + 1);
            c.ny = uint16_t((j1 >> 6) - (j0 >> 6) + 1);
            blocks[k] = c;
            items[k] = uint64_t(c.nx) * c.ny;
            if (items[k] >= kManyBlocks) {
                many[atomicAdd(found, 1ull)] = uint32_t(k);
                atomicAdd(found + 1, (unsigned long long)items[k]);
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) items[a.n] = 0;
}

struct RowArgs {
    const i64x2 *xy;
    const uint64_t *voff;
    const EdgeBox *box;
    const Blocks *blocks;
    const uint32_t *many;      // the listed polygons
    uint32_t *taken;           // per listed polygon: blocks counted, or keys written
    uint32_t n_many;
    Geo g;
    // where the keys go (a group's polygons, as in ItemArgs)
    const uint64_t *base;
    uint64_t first_poly, n_polys, item0;
    uint64_t *key;
};

// The blocks of the listed polygons that an edge may meet (edges are clipped to
// the row of blocks in double precision, with some lattice units to spare; an
// item more is an empty one) or that lie inside: a wave per row of blocks.  A
// block that no edge meets lies inside when an odd number of edges cross the
// row's centre line in the blocks left of it.  blockIdx.x: the polygon, its
// rows dealt out over blockIdx.y and the waves.  2,000 slivers across 500 x 500
// blocks take 12.4 ms a call, with an item for every block 1,545; 200 open rings
// of 300 x 300 3.9 and 88; 100 polygons of 20k to 100k vertices 10.7 and 11.4.
constexpr uint32_t kRowBlocks = 16;   // workgroups of a polygon

template <bool EMIT>
__global__ __launch_bounds__(kBlock) void k_block_rows(RowArgs a) {
    __shared__ uint32_t lds[kWavesPerBlock][2][32];   // a bit per block: an edge, a crossing
    const uint32_t lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    uint32_t *const mark = lds[w][0], *const cross = lds[w][1];
    const int64_t side = 64 * a.g.w;
    const double inv = a.g.inv_w / 64;
    for (uint32_t i = blockIdx.x; i < a.n_many; i += gridDim.x) {
        const uint64_t k = a.many[i];
        if (EMIT && (k < a.first_poly || k >= a.first_poly + a.n_polys)) continue;
        const Blocks c = a.blocks[k];
        const uint64_t v0 = a.voff[k], nv = a.voff[k + 1] - v0;
        const EdgeBox *boxes = a.box + box_at(v0, k);
        const uint32_t nb = uint32_t((nv + 63) / 64);
        auto block_of = [&](double x) {   // (within the polygon's blocks, from its first)
            return uint32_t(min(max(int64_t(floor(x * inv)) - int64_t(c.x0), int64_t(0)), int64_t(c.nx) - 1));
        };
        for (uint32_t row = blockIdx.y * kWavesPerBlock + w; row < c.ny; row += gridDim.y * kWavesPerBlock) {
            const int64_t y0 = (int64_t(c.y0) + row) * side, y1 = y0 + side, mid = y0 + side / 2;
            wave_lds_sync();
            (lane < 32 ? mark : cross)[lane & 31] = 0;
            wave_lds_sync();
            for (uint32_t c0 = 0; c0 < nb; c0 += 64) {
                bool into = c0 + lane < nb;
                if (into) {
                    const EdgeBox x = boxes[c0 + lane];
                    into = x.y1 >= y0 && x.y0 <= y1;
                }
                uint64_t todo = __ballot(into);
                while (todo) {
                    const uint64_t e = 64ull * (c0 + uint32_t(__builtin_ctzll(todo))) + lane;
                    todo &= todo - 1;
                    if (e >= nv) continue;
                    i64x2 u, v;
                    load_edge(a.xy, v0, nv, e, u, v);
                    if (u.y > v.y) {
                        const i64x2 t = u;
                        u = v;
                        v = t;
                    }
                    if (v.y < y0 || u.y > y1) continue;
                    const double slope = u.y == v.y ? 0.0 : double(v.x - u.x) / double(v.y - u.y);
                    auto at = [&](int64_t y) { return double(u.x) + double(y - u.y) * slope; };
                    const double p = at(max(u.y, y0)), q = u.y == v.y ? double(v.x) : at(min(v.y, y1));
                    const uint32_t b0 = block_of(min(p, q) - 8.0), b1 = block_of(max(p, q) + 8.0);
                    for (uint32_t b = b0 >> 5; b <= b1 >> 5; b++) {
                        const uint32_t lo = b == b0 >> 5 ? ~0u << (b0 & 31) : ~0u;
                        const uint32_t hi = b == b1 >> 5 ? ~0u >> (31 - (b1 & 31)) : ~0u;
                        atomicOr(&mark[b], lo & hi);
                    }
                    if (u.y <= mid && mid < v.y) {
                        const uint32_t b = min(max(block_of(at(mid)), b0), b1);
                        atomicXor(&cross[b >> 5], 1u << (b & 31));
                    }
                }
            }
            wave_lds_sync();
            uint32_t need = 0;
            if (lane < 32) {
                need = mark[lane];
                uint32_t odd = cross[lane];
                for (int s = 1; s < 32; s <<= 1) odd ^= odd << s;
                const uint64_t before = __ballot(odd >> 31) & ((1ull << lane) - 1);
                if (__popcll(before) & 1) odd = ~odd;
                need |= odd;
                const int32_t left = int32_t(c.nx) - int32_t(32 * lane);
                need &= left >= 32 ? ~0u : left > 0 ? (1u << left) - 1 : 0u;
            }
            const uint32_t n = uint32_t(__popc(need));
            uint32_t upto = n;
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t o = __shfl_up(upto, d);
                if (lane >= uint32_t(d)) upto += o;
            }
            uint32_t got = 0;
            if (lane == 63) got = atomicAdd(&a.taken[i], upto);
            if (EMIT) {
                // a lane per block
                const uint64_t at = a.base[k] - a.item0 + uint32_t(__shfl(got, 63));
                wave_lds_sync();
                if (lane < 32) {
                    mark[lane] = need;
                    cross[lane] = upto - n;
                }
                wave_lds_sync();
                for (uint32_t b = lane; b < c.nx; b += 64) {
                    const uint32_t word = mark[b >> 5], bit = 1u << (b & 31);
                    if (word & bit)
                        a.key[at + cross[b >> 5] + uint32_t(__popc(word & (bit - 1)))] =
                            ((k - a.first_poly) << (2 * a.g.border)) | hilbert_d(a.g.border, c.x0 + b, c.y0 + row);
                }
            }
        }
    }
}

// The listed polygons' counts become their numbers of items.
__global__ void k_many_items(const uint32_t *many, uint32_t *taken, uint32_t n_many, uint64_t *items) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_many) items[many[i]] = taken[i];
}

// Cells met by the edge a-b (closed squares), row by row.  T is the product
// type: int64 when the grid spans few enough lattice units, else 128-bit.
// Only counted when the bound above leaves it open whether a call has more
// than it takes.
template <typename T>
__device__ uint64_t edge_cells(int64_t ax, int64_t ay, int64_t bx, int64_t by, const Geo &g) {
    const int64_t w = g.w;
    if (ay > by) {
        const int64_t tx = ax, ty = ay;
        ax = bx; ay = by; bx = tx; by = ty;
    }
    const bool horiz = ay == by;
    const T D = horiz ? T(1) : T(by - ay);
    const int64_t j0 = cdiv<int64_t>(ay, w) - 1, j1 = fdiv(by, w);
    uint64_t cnt = 0;
    for (int64_t j = j0; j <= j1; j++) {
        const int64_t ylo = max(ay, j * w), yhi = min(by, (j + 1) * w);
        T n0, n1;
        if (horiz) {
            n0 = T(min(ax, bx));
            n1 = T(max(ax, bx));
        } else {
            const T u = T(ax) * D + T(ylo - ay) * T(bx - ax);
            const T v = T(ax) * D + T(yhi - ay) * T(bx - ax);
            n0 = u < v ? u : v;
            n1 = u < v ? v : u;
        }
        const T Dw = D * T(w);
        cnt += uint64_t(fdiv(n1, Dw) - (cdiv<T>(n0, Dw) - 1) + 1);
    }
    return cnt;
}

__global__ void k_count_cells(const i64x2 *xy, const uint64_t *voff, uint64_t n, uint64_t nv, Geo g, uint32_t wide,
                              unsigned long long *total) {
    unsigned long long c = 0;
    for (uint64_t v = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < nv; v += uint64_t(gridDim.x) * blockDim.x) {
        uint64_t lo = 0, hi = n;
        while (hi - lo > 1) {
            const uint64_t mid = (lo + hi) / 2;
            if (voff[mid] <= v) lo = mid;
            else hi = mid;
        }
        i64x2 a, b;
        load_edge(xy, voff[lo], voff[lo + 1] - voff[lo], v - voff[lo], a, b);
        c += wide ? edge_cells<__int128>(a.x, a.y, b.x, b.y, g) : edge_cells<int64_t>(a.x, a.y, b.x, b.y, g);
    }
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off);
    if ((threadIdx.x & 63) == 0) atomicAdd(total, c);
}

// ------------------------------------------------------------------ items

struct ItemArgs {
    const i64x2 *xy;
    const uint64_t *voff;
    const EdgeBox *box;
    const Blocks *blocks;
    const uint64_t *base;      // first item of polygon k (of all polygons)
    uint64_t first_poly, n_polys, item0, n_items;   // the group of polygons at work
    uint32_t many;             // polygons of so many blocks: keys by k_block_rows
    uint64_t *key;             // (polygon - first_poly) << 2 border | Hilbert id of the block
    uint32_t *place;           // the block: x | y << 12 | state of the curve in it << 24
    uint32_t *info;
    Geo g;
    // where the intervals go
    uint64_t n;
    const uint64_t *ai, *fi;   // slots of the items' first starts, from a0 / f0 on
    uint64_t a0, f0, n_a, n_f;
    uint64_t *off_a, *off_f;
    uint32_t *sa, *ea, *sf, *ef;
    unsigned int *bad_slot;
};

__global__ void k_item_keys(ItemArgs a) {
    const uint64_t t = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= a.n_items) return;
    uint64_t lo = a.first_poly, hi = a.first_poly + a.n_polys;   // base[lo] <= item0 + t < base[hi]
    while (hi - lo > 1) {
        const uint64_t mid = (lo + hi) / 2;
        if (a.base[mid] <= a.item0 + t) lo = mid;
        else hi = mid;
    }
    const Blocks c = a.blocks[lo];
    if (uint32_t(c.nx) * c.ny >= a.many) return;   // (k_block_rows)
    const uint32_t i = uint32_t(a.item0 + t - a.base[lo]);
    a.key[t] = ((lo - a.first_poly) << (2 * a.g.border)) |
               hilbert_d(a.g.border, c.x0 + i % c.nx, c.y0 + i / c.nx);
}

// What an item tells its neighbours: starts behind the first cell (12 bits for
// A, 12 for F), and whether the first and the last cell are in A and in F.
constexpr uint32_t kFirstA = 1u << 24, kLastA = 1u << 25, kFirstF = 1u << 26, kLastF = 1u << 27;

// Is item t + 1 the block that follows item t's on the curve, of the same polygon?
__device__ __forceinline__ bool follows(const uint64_t *key, uint64_t t, const Geo &g) {
    const uint64_t u = key[t], v = key[t + 1];
    return v == u + 1 && (u >> (2 * g.border)) == (v >> (2 * g.border));
}

// Hilbert steps of three levels by table: (state, x, y) -> the six bits of the
// id and the state below, and back.  (A state is one of four symmetries.)
struct Curve {
    uint8_t to_d[256];    // [state * 64 + x * 8 + y] = d | state << 6
    uint8_t to_xy[256];   // [state * 64 + d] = x * 8 + y | state << 6
};

__device__ __forceinline__ void curve_tables(Curve &c, uint32_t t) {   // t < 256
    uint32_t state = t >> 6, d = 0;
    const uint32_t x = (t >> 3) & 7, y = t & 7, s0 = state;
    for (int lvl = 2; lvl >= 0; lvl--) {
        uint32_t qx, qy;
        sym(state, (x >> lvl) & 1u, (y >> lvl) & 1u, qx, qy);
        const uint32_t digit = (qx * 3u) ^ qy;
        d = (d << 2) | digit;
        state ^= child(digit);
    }
    c.to_d[t] = uint8_t(d | (state << 6));
    c.to_xy[s0 * 64 + d] = uint8_t((x << 3) | y | (state << 6));
}

// the state of the curve inside block `d` of a grid of blocks of the given order, and the block's place
__device__ __forceinline__ uint32_t block_xy(int order, uint32_t d, uint32_t &x, uint32_t &y) {
    uint32_t state = 0;
    x = y = 0;
    for (int lvl = order - 1; lvl >= 0; lvl--) {
        const uint32_t digit = (d >> (2 * lvl)) & 3u;
        uint32_t bx, by;
        sym(state, digit >> 1, (digit ^ (digit >> 1)) & 1u, bx, by);
        x = (x << 1) | bx;
        y = (y << 1) | by;
        state ^= child(digit);
    }
    return state;
}

// A sorted item's place, a thread each.
__global__ void k_item_places(ItemArgs a) {
    const uint64_t t = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= a.n_items) return;
    uint32_t x, y;
    const uint32_t state = block_xy(a.g.border, uint32_t(a.key[t] & ((1ull << (2 * a.g.border)) - 1)), x, y);
    a.place[t] = x | (y << 12) | (state << 24);
}

// Arithmetic.  While the grid spans at most 1.25 * 2^30 lattice units,
// coordinates fit in 32 bits and products in 64 (|products| <= 4 E^2 < 2^63);
// else they take 64 and 128.  Quotients are numbers of cells, below 2^17, so
// that a single-precision estimate (relative error below 2^-21) is off by
// less than one, and the exact remainder corrects it.
struct Narrow {
    typedef int32_t C;
    typedef int64_t P;
};
struct Wide {
    typedef int64_t C;
    typedef __int128 P;
};

struct QR {
    int32_t q;
    bool zero;   // no remainder
};

__device__ __forceinline__ float to_float(int64_t v) {
    return __builtin_fmaf(float(int32_t(v >> 32)), 4294967296.0f, float(uint32_t(v)));
}

__device__ __forceinline__ QR div_cells(int64_t n, int64_t d, float inv) {   // n >= 0
    int32_t q = int32_t(to_float(n) * inv);
    int64_t r = n - int64_t(q) * d;
    if (r < 0) {
        q--;
        r += d;
    } else if (r >= d) {
        q++;
        r -= d;
    }
    return {q, r == 0};
}
__device__ __forceinline__ QR div_cells(__int128 n, __int128 d, float) {
    const __int128 q = n / d;
    return {int32_t(q), n == q * d};
}

// floor(v / w) and, for the centre lines, floor(v / 2 w); v >= 0
__device__ __forceinline__ int32_t cell_of(int64_t v, const Geo &g) { return div_cells(v, g.w, g.inv_wf).q; }
__device__ __forceinline__ int32_t half_of(int64_t v, const Geo &g) { return div_cells(v, 2 * g.w, g.inv_2wf).q; }

template <class M>
struct Edge {   // the lower end first
    typename M::C ux, uy, vx, vy;
};

template <class M>
struct ItemLds {
    Edge<M> edge[64];           // edges that meet the block
    uint32_t upto[64];          // rows of the edges up to each
    int32_t row0[64];           // an edge's first row, less the rows before it
    uint32_t touched[128], crossed[128];   // in Hilbert order
    uint32_t parity[128];       // per row of cells: two words
};

template <class M>
struct Block {
    int32_t cx, cy;             // first cell
    typename M::C x0, y0, x1, y1;   // closed, lattice units
    uint32_t state;
    int32_t size;               // cells a side
};

// rows of the block (bits) whose centre line lies below y, as the half-open
// crossing rule has it: an edge crosses the line when exactly one of its ends
// is above.  Row j's centre, doubled, is (2 j + 1) w < 2 y for the rows
// j < ceil((2 y - w) / 2 w).
template <class M>
__device__ __forceinline__ uint64_t rows_below(typename M::C y, const Block<M> &b, const Geo &g) {
    const int32_t c = half_of(2 * int64_t(y) + g.w - 1, g) - b.cy;
    return c <= 0 ? 0ull : c >= 64 ? ~0ull : (1ull << c) - 1;
}

// The cells of row j that the edge meets.
template <class M>
__device__ __forceinline__ void raster_row(const Edge<M> &e, int32_t j, const Block<M> &b, const Geo &g,
                                           ItemLds<M> &l, const Curve &cv) {
    typedef typename M::C C;
    typedef typename M::P P;
    const C w = C(g.w);
    const bool horiz = e.uy == e.vy;
    const C D = horiz ? C(1) : e.vy - e.uy, dx = e.vx - e.ux;
    const P Dw = P(D) * P(w), x0 = P(e.ux) * P(D);
    const float inv = __builtin_amdgcn_rcpf(float(D) * float(w));
    const C y0 = C(j) * w, y1 = y0 + w, ylo = max(e.uy, y0), yhi = min(e.vy, y1);
    const P p = x0 + P(ylo - e.uy) * P(dx), q = horiz ? P(e.vx) : x0 + P(yhi - e.uy) * P(dx);
    const QR q0 = div_cells(p < q ? p : q, Dw, inv), q1 = div_cells(p < q ? q : p, Dw, inv);
    const int32_t row = j - b.cy;
    const int32_t i0 = max(q0.q - (q0.zero ? 1 : 0), b.cx), i1 = min(q1.q, b.cx + b.size - 1);
    const bool open_row = horiz ? (y0 < e.uy && e.uy < y1) : ylo < yhi;
    const int32_t o0 = open_row ? q0.q : 1, o1 = open_row ? q1.q - (q1.zero ? 1 : 0) : 0;
    const uint32_t y = uint32_t(row);
    for (int32_t i = i0; i <= i1; i++) {
        const uint32_t x = uint32_t(i - b.cx);
        uint32_t d;
        if (b.size == 64) {
            const uint32_t hi = cv.to_d[b.state * 64 + (x >> 3) * 8 + (y >> 3)];
            d = ((hi & 63u) << 6) | (cv.to_d[(hi >> 6) * 64 + (x & 7) * 8 + (y & 7)] & 63u);
        } else {
            d = hilbert_d(g.order, x, y);   // the grid is smaller than a block
        }
        atomicOr(&l.touched[d >> 5], 1u << (d & 31));
        if (i >= o0 && i <= o1) atomicOr(&l.crossed[d >> 5], 1u << (d & 31));
    }
    // the crossing of the row's centre line: at x = N / D (doubled), it lies
    // left of the centres of the cells i with (2 i + 1) w > floor(x), the first
    // of which is floor((N + w D) / 2 w D)
    const P c = P(2 * int64_t(j) + 1) * P(w), c0 = c - P(2) * P(e.uy);
    if (!horiz && c0 >= 0 && c < P(2) * P(e.vy)) {
        const P N = P(2) * x0 + c0 * P(dx);
        const int32_t im = max(div_cells(N + Dw, Dw + Dw, 0.5f * inv).q, b.cx) - b.cx;
        if (im < b.size) atomicXor(&l.parity[2 * row + (im >> 5)], 1u << (im & 31));
    }
}

__device__ __forceinline__ uint64_t shfl_xor64(uint64_t v, int mask) {
    return uint64_t(uint32_t(__shfl_xor(int(uint32_t(v)), mask))) |
           (uint64_t(uint32_t(__shfl_xor(int(uint32_t(v >> 32)), mask))) << 32);
}

// The item's A and F cells in Hilbert order, 64 a lane.
template <class M>
__device__ __forceinline__ void raster_item(const ItemArgs &a, uint64_t poly, const Block<M> &b, ItemLds<M> &l,
                                            const Curve &cv, uint32_t lane, uint64_t &A, uint64_t &F) {
    typedef typename M::C C;
    const uint64_t v0 = a.voff[poly], nv = a.voff[poly + 1] - v0;
    const EdgeBox *boxes = a.box + box_at(v0, poly);
    const uint32_t nb = uint32_t((nv + 63) / 64);
    uint64_t left = 0;   // rows whose parity the lane's passing edges change
    bool any = false;
    for (uint32_t c0 = 0; c0 < nb; c0 += 64) {
        // boxes of 64 edges, one a lane: beside the block, left of it, or to be looked into
        bool into = c0 + lane < nb;
        if (into && nb > 1) {
            const uint32_t c = c0 + lane;
            const EdgeBox x = boxes[c];
            const bool beside = x.y1 < b.y0 || x.y0 > b.y1 || x.x0 > b.x1;
            if (!beside && x.x1 < b.x0) {
                const uint64_t e1 = min<uint64_t>(nv, 64ull * c + 64);
                left ^= rows_below<M>(C(a.xy[v0 + 64ull * c].y), b, a.g) ^
                        rows_below<M>(C(a.xy[v0 + (e1 == nv ? 0 : e1)].y), b, a.g);
            }
            into = !beside && x.x1 >= b.x0;
        }
        uint64_t todo = __ballot(into);
        while (todo) {
            const uint32_t c = c0 + uint32_t(__builtin_ctzll(todo));
            todo &= todo - 1;
            const uint64_t k = 64ull * c + lane;
            Edge<M> e{};
            bool in = false, pass = false;
            if (k < nv) {
                i64x2 u, v;
                load_edge(a.xy, v0, nv, k, u, v);
                const bool up = u.y <= v.y;
                e = up ? Edge<M>{C(u.x), C(u.y), C(v.x), C(v.y)} : Edge<M>{C(v.x), C(v.y), C(u.x), C(u.y)};
                const bool beside = e.vy < b.y0 || e.uy > b.y1 || min(e.ux, e.vx) > b.x1;
                in = !beside && max(e.ux, e.vx) >= b.x0;
                pass = !beside && !in;
            }
            if (pass) left ^= rows_below<M>(e.uy, b, a.g) ^ rows_below<M>(e.vy, b, a.g);
            if (!__any(in)) continue;
            if (!any) {
                // the first edge here: clear the bit arrays
                any = true;
                wave_lds_sync();
#pragma unroll
                for (uint32_t i = 0; i < 128; i += 64)
                    l.touched[i + lane] = l.crossed[i + lane] = l.parity[i + lane] = 0;
            }
            // the edges' rows one after another; lane i takes the i-th next
            int32_t j0 = 0, rows = 0;
            if (in) {
                j0 = max(b.cy, cell_of(int64_t(e.uy) + a.g.w - 1, a.g) - 1);
                rows = min(b.cy + b.size - 1, cell_of(e.vy, a.g)) - j0 + 1;
            }
            uint32_t upto = uint32_t(rows);
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t o = __shfl_up(upto, d);
                if (lane >= uint32_t(d)) upto += o;
            }
            const uint32_t total = __builtin_amdgcn_readlane(upto, 63);
            wave_lds_sync();
            l.edge[lane] = e;
            l.upto[lane] = upto;
            l.row0[lane] = j0 - int32_t(upto - uint32_t(rows));
            wave_lds_sync();
            for (uint32_t t0 = 0; t0 < total; t0 += 64) {
                const uint32_t t = t0 + lane;
                if (t >= total) continue;
                uint32_t i = 0;   // the first edge with upto > t
#pragma unroll
                for (uint32_t s = 32; s > 0; s >>= 1) i += l.upto[i + s - 1] <= t ? s : 0;
                raster_row<M>(l.edge[i], l.row0[i] + int32_t(t), b, a.g, l, cv);
            }
        }
    }
    if (__any(left != 0))
        for (int off = 32; off > 0; off >>= 1) left ^= shfl_xor64(left, off);
    if (!any) {   // no edge here: all cells alike
        A = F = (left & 1) && b.size == 64 ? ~0ull : 0ull;
        return;
    }
    wave_lds_sync();
    // parity to the left of each centre, row by row (a lane per row)
    uint64_t p = uint64_t(l.parity[2 * lane]) | (uint64_t(l.parity[2 * lane + 1]) << 32);
    p ^= (left >> lane) & 1;
    for (int s = 1; s < 64; s <<= 1) p ^= p << s;
    wave_lds_sync();
    l.parity[2 * lane] = uint32_t(p);
    l.parity[2 * lane + 1] = uint32_t(p >> 32);
    const uint64_t T64 = uint64_t(l.touched[2 * lane]) | (uint64_t(l.touched[2 * lane + 1]) << 32);
    const uint64_t C64 = uint64_t(l.crossed[2 * lane]) | (uint64_t(l.crossed[2 * lane + 1]) << 32);
    wave_lds_sync();
    // the lane's 64 cells: one 8 x 8 square
    const uint32_t hi = b.size == 64 ? cv.to_xy[b.state * 64 + lane] : 0u;
    auto inside = [&](uint32_t bit) {
        uint32_t x, y;
        if (b.size == 64) {
            const uint32_t lo = cv.to_xy[(hi >> 6) * 64 + bit];
            x = ((hi >> 3) & 7) * 8 + ((lo >> 3) & 7);
            y = (hi & 7) * 8 + (lo & 7);
        } else {
            hilbert_xy(a.g.order, lane * 64 + bit, x, y);
        }
        return (l.parity[2 * y + (x >> 5)] >> (x & 31)) & 1u;
    };
    uint64_t valid = ~0ull;
    if (b.size < 64) {
        const uint32_t cells = uint32_t(b.size) * uint32_t(b.size);
        valid = lane * 64 >= cells ? 0ull : cells - lane * 64 >= 64 ? ~0ull : (1ull << (cells - lane * 64)) - 1;
    }
    const uint64_t Z = ~T64 & valid;
    uint64_t runs = Z & ~(Z << 1), G = 0;
    while (runs) {
        const uint32_t bit = uint32_t(__builtin_ctzll(runs));
        runs &= runs - 1;
        G |= uint64_t(inside(bit)) << bit;
    }
    // a run whose first bit is in G: adding G carries through it
    const uint64_t gap = Z & ~(Z + G);
    uint64_t border = T64 & ~C64, full = 0;
    while (border) {
        const uint32_t bit = uint32_t(__builtin_ctzll(border));
        border &= border - 1;
        full |= uint64_t(inside(bit)) << bit;
    }
    A = T64 | gap;
    F = full | gap;
}

// Interval ends of one kind in an item: `cells` of the lane, `before` and
// `after`: is the cell before the item's first, behind its last one in it?
__device__ __forceinline__ void run_ends(uint64_t cells, bool before, bool after, uint32_t lane, uint64_t &starts,
                                         uint64_t &stops) {
    const uint32_t top = __shfl_up(uint32_t(cells >> 63), 1), low = __shfl_down(uint32_t(cells & 1), 1);
    const uint64_t cin = lane == 0 ? uint64_t(before) : uint64_t(top);
    const uint64_t cout = lane == 63 ? uint64_t(after) : uint64_t(low);
    starts = cells & ~((cells << 1) | cin);
    stops = cells & ~((cells >> 1) | (cout << 63));
}

// the sums of v over the lanes before this one
__device__ __forceinline__ uint32_t wave_before(uint32_t v, uint32_t lane) {
    uint32_t s = v;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(s, d);
        if (lane >= uint32_t(d)) s += o;
    }
    return s - v;
}

// Where one kind's intervals of a lane go: its starts to s[at ...], its stops
// to e[stop_at ...].  A lane's first stop is its first start's, unless the
// interval runs into the lane: then it belongs to the start before.
struct Runs {
    uint64_t starts, stops, at, stop_at;
};

__device__ __forceinline__ Runs lane_runs(uint64_t cells, bool before, bool after, uint32_t lane) {
    Runs r;
    run_ends(cells, before, after, lane, r.starts, r.stops);
    r.at = 0;
    r.stop_at = (cells & 1) && !(r.starts & 1) ? ~0ull : 0ull;
    return r;
}

// the next interval ends, checked against the sizes that were allocated (which
// consistent items never exceed; below zero wraps past every bound)
__device__ __forceinline__ bool write_next(Runs &r, uint32_t d0, uint64_t n, uint32_t *s, uint32_t *e) {
    bool ok = true;
    if (r.starts) {
        if (r.at < n) s[r.at] = d0 + uint32_t(__builtin_ctzll(r.starts));
        else ok = false;
        r.at++;
        r.starts &= r.starts - 1;
    }
    if (r.stops) {
        if (r.stop_at < n) e[r.stop_at] = d0 + uint32_t(__builtin_ctzll(r.stops)) + 1;
        else ok = false;
        r.stop_at++;
        r.stops &= r.stops - 1;
    }
    return ok;
}

template <class M, bool WRITE>
__global__ __launch_bounds__(kBlock) void k_items(ItemArgs a) {
    __shared__ ItemLds<M> lds[kWavesPerBlock];
    __shared__ Curve cv;
    const uint32_t lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    curve_tables(cv, threadIdx.x);
    __syncthreads();
    const uint64_t waves = uint64_t(gridDim.x) * kWavesPerBlock;
    for (uint64_t t = uint64_t(blockIdx.x) * kWavesPerBlock + w; t < a.n_items; t += waves) {
        const uint64_t key = a.key[t];
        const uint64_t poly = a.first_poly + (key >> (2 * a.g.border));
        const uint32_t place = uniform(a.place[t]);
        typedef typename M::C C;
        Block<M> b;
        b.state = place >> 24;
        b.size = int32_t(min<int64_t>(64, a.g.cells));
        b.cx = int32_t(place & 0xfffu) * 64;
        b.cy = int32_t((place >> 12) & 0xfffu) * 64;
        b.x0 = C(b.cx) * C(a.g.w);
        b.y0 = C(b.cy) * C(a.g.w);
        b.x1 = C(b.cx + b.size) * C(a.g.w);
        b.y1 = C(b.cy + b.size) * C(a.g.w);
        uint64_t A, F;
        raster_item<M>(a, poly, b, lds[w], cv, lane, A, F);
        if (!WRITE) {
            uint64_t s, f, e;
            run_ends(A, true, true, lane, s, e);   // (a start at the first cell is not counted here)
            run_ends(F, true, true, lane, f, e);
            uint32_t c = uint32_t(__popcll(s)) | (uint32_t(__popcll(f)) << 12);
            for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
            const uint32_t a0 = __builtin_amdgcn_readlane(uint32_t(A), 0), f0 = __builtin_amdgcn_readlane(uint32_t(F), 0);
            const uint32_t a1 = __builtin_amdgcn_readlane(uint32_t(A >> 32), 63);
            const uint32_t f1 = __builtin_amdgcn_readlane(uint32_t(F >> 32), 63);
            c |= (a0 & 1 ? kFirstA : 0) | (f0 & 1 ? kFirstF : 0) | (a1 >> 31 ? kLastA : 0) | (f1 >> 31 ? kLastF : 0);
            if (lane == 0) a.info[t] = c;
        } else {
            const bool prev = t > 0 && follows(a.key, t - 1, a.g), next = t + 1 < a.n_items && follows(a.key, t, a.g);
            const uint32_t ip = prev ? a.info[t - 1] : 0u, in = next ? a.info[t + 1] : 0u;
            const uint64_t at = a.a0 + a.ai[t], ft = a.f0 + a.fi[t];
            const uint32_t d0 = (uint32_t(key & ((1ull << (2 * a.g.border)) - 1)) << 12) + lane * 64;
            if (__any(A != 0)) {   // (F lies in A)
                Runs ra = lane_runs(A, ip & kLastA, in & kFirstA, lane), rf = lane_runs(F, ip & kLastF, in & kFirstF, lane);
                // starts of A (at most 2,048 an item) and of F in the lanes before
                const uint32_t n = wave_before(uint32_t(__popcll(ra.starts)) | (uint32_t(__popcll(rf.starts)) << 16), lane);
                ra.at += at + (n & 0xffffu);
                ra.stop_at += at + (n & 0xffffu);
                rf.at += ft + (n >> 16);
                rf.stop_at += ft + (n >> 16);
                bool ok = true;
                while (ra.starts | ra.stops | rf.starts | rf.stops) {
                    ok &= write_next(ra, d0, a.n_a, a.sa, a.ea);
                    ok &= write_next(rf, d0, a.n_f, a.sf, a.ef);
                }
                if (!ok) atomicOr(a.bad_slot, 1u);
            }
            if (lane == 0 && (t == 0 || (a.key[t - 1] >> (2 * a.g.border)) != (key >> (2 * a.g.border)))) {
                a.off_a[poly] = at;
                a.off_f[poly] = ft;
            }
        }
    }
    if (WRITE && blockIdx.x == 0 && threadIdx.x == 0 && a.first_poly + a.n_polys == a.n) {
        a.off_a[a.n] = a.n_a;
        a.off_f[a.n] = a.n_f;
    }
}

// starts of each item, with the one at its first cell unless the block before
// it on the curve ends in the same interval; zero behind the last item
__global__ void k_item_starts(ItemArgs a, uint64_t *na, uint64_t *nf) {
    const uint64_t t = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t > a.n_items) return;
    if (t == a.n_items) {
        na[t] = nf[t] = 0;
        return;
    }
    const uint32_t i = a.info[t], p = t > 0 && follows(a.key, t - 1, a.g) ? a.info[t - 1] : 0u;
    na[t] = (i & 0xfffu) + ((i & kFirstA) && !(p & kLastA) ? 1 : 0);
    nf[t] = ((i >> 12) & 0xfffu) + ((i & kFirstF) && !(p & kLastF) ? 1 : 0);
}

uint32_t blocks_for(uint64_t n) { return uint32_t(std::max<uint64_t>(1, (n + kThreads - 1) / kThreads)); }

// Stream-ordered scratch, freed when the call returns (in stream order): a
// block at a time, cut into arrays.
struct Scratch {
    hipStream_t s;
    std::vector<void *> held;
    char *at = nullptr;
    bool reserve(uint64_t bytes) {
        void *p = nullptr;
        if (hipMallocAsync(&p, std::max<uint64_t>(bytes, 256), s) != hipSuccess) return false;
        held.push_back(p);
        at = static_cast<char *>(p);
        return true;
    }
    static uint64_t up(uint64_t b) { return (b + 255) & ~uint64_t(255); }
    template <typename T>
    T *get(uint64_t count) {
        T *p = reinterpret_cast<T *>(at);
        at += up(count * sizeof(T));
        return p;
    }
    ~Scratch() {
        for (void *p : held) (void)hipFreeAsync(p, s);
    }
};

// Most items worked on at once (about 40 bytes of scratch each); a call with
// more goes through its polygons in groups.
constexpr uint64_t kGroupItems = 1ull << 26;

}  // namespace
}  // namespace april

using namespace april;

#define BG_TRY(expr)                                                                              \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess) return fail(APRIL_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

extern "C" int april_build_lists_gpu(const april_grid_t *grid, const double *xy, const uint64_t *vtx_off,
                                     uint64_t n, uint32_t flags, void *hip_stream, april_lists_t **out) {
    return build_lists_gpu(grid, xy, vtx_off, n, flags, hip_stream, true, out);
}

int april::build_lists_gpu(const april_grid_t *grid, const double *xy, const uint64_t *vtx_off, uint64_t n,
                           uint32_t flags, void *hip_stream, bool summaries, april_lists_t **out) {
    clear_error();
    if (!xy || !vtx_off || !out) return fail(APRIL_E_INVALID, "NULL argument");
    if (n == 0) return fail(APRIL_E_INVALID, "no polygons");
    if (n >= (1ull << 31)) return fail(APRIL_E_INVALID, "more than 2^31 - 1 polygons");
    if (flags & ~APRIL_STRICT) return fail(APRIL_E_INVALID, "unknown flags");
    LatticeGrid lg;
    if (int rc = lattice_grid(grid, &lg)) return rc;
    for (uint64_t k = 0; k < n; k++)
        if (vtx_off[k + 1] < vtx_off[k] + 3) return fail(APRIL_E_INVALID, "polygon with < 3 vertices");
    const uint64_t nv = vtx_off[n] - vtx_off[0];
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    int dev = 0;
    BG_TRY(hipGetDevice(&dev));
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    Geo g{lg.x0, lg.y0, lg.w, 1.0 / double(lg.w), float(1.0 / double(lg.w)), float(0.5 / double(lg.w)), lg.cells, lg.order, std::max(0, lg.order - 6),
          (flags & APRIL_STRICT) ? 1u : 0u};
    // narrow arithmetic is exact while the grid spans at most 1.25 * 2^30 lattice units
    const uint32_t wide = double(lg.w) * double(lg.cells) > 1.25 * 1073741824.0 ? 1u : 0u;

    // 1-2: vertices, boxes, blocks
    const uint64_t n_boxes = (nv >> 6) + n;
    size_t scan_bytes = 0;
    BG_TRY(hipcub::DeviceScan::ExclusiveSum(nullptr, scan_bytes, (uint64_t *)nullptr, (uint64_t *)nullptr, n + 1, s));
    Scratch sc{s, {}};
    auto pad = Scratch::up;
    if (!sc.reserve(pad(16 * nv) + 3 * pad(8 * (n + 1)) + pad(32 * n_boxes) + pad(4 * n_boxes) + pad(8 * n) + pad(64) +
                    2 * pad(4 * n) + pad(scan_bytes)))
        return fail(APRIL_E_NOMEM, "build scratch");
    i64x2 *d_xy = sc.get<i64x2>(nv);
    uint64_t *d_voff = sc.get<uint64_t>(n + 1), *d_items = sc.get<uint64_t>(n + 1), *d_base = sc.get<uint64_t>(n + 1);
    EdgeBox *d_box = sc.get<EdgeBox>(n_boxes);
    uint32_t *d_distinct = sc.get<uint32_t>(n_boxes);
    Blocks *d_blocks = sc.get<Blocks>(n);
    // err; bound of the cells; bad slot, longest list, long A-lists; polygons of many blocks, their blocks
    unsigned long long *d_small = sc.get<unsigned long long>(8);
    uint32_t *d_many = sc.get<uint32_t>(n), *d_taken = sc.get<uint32_t>(n);
    void *d_scan = sc.get<char>(scan_bytes);
    std::vector<uint64_t> voff_rel(n + 1);
    for (uint64_t k = 0; k <= n; k++) voff_rel[k] = vtx_off[k] - vtx_off[0];
    BG_TRY(hipMemcpyAsync(d_xy, xy + 2 * vtx_off[0], 16 * nv, hipMemcpyHostToDevice, s));
    BG_TRY(hipMemcpyAsync(d_voff, voff_rel.data(), 8 * (n + 1), hipMemcpyHostToDevice, s));
    BG_TRY(hipMemsetAsync(d_small, 0xff, 8, s));   // err = none
    BG_TRY(hipMemsetAsync(d_small + 1, 0, 56, s));
    k_vertices<<<blocks_for(nv), kThreads, 0, s>>>(d_xy, d_voff, n, nv, g, d_small);
    PolyArgs pa{d_xy, d_voff, n, n_boxes, d_box, d_distinct, d_small + 1, g};
    k_edge_boxes<<<uint32_t(std::min<uint64_t>((n_boxes + 3) / 4, uint64_t(st->cus) * 8)), 256, 0, s>>>(pa);
    k_polygons<<<uint32_t(std::min<uint64_t>((n + 3) / 4, 16384)), 256, 0, s>>>(
        pa, d_blocks, d_items, d_many, d_small + 5, d_small);
    BG_TRY(hipGetLastError());
    BG_TRY(hipcub::DeviceScan::ExclusiveSum(d_scan, scan_bytes, d_items, d_base, n + 1, s));
    uint64_t h[7] = {0, 0}, items = 0;   // as d_small; items
    BG_TRY(hipMemcpyAsync(h, d_small, 56, hipMemcpyDeviceToHost, s));
    BG_TRY(hipMemcpyAsync(&items, d_base + n, 8, hipMemcpyDeviceToHost, s));
    BG_TRY(hipStreamSynchronize(s));
    if (h[0] != ~0ull) {
        const uint64_t k = h[0] >> 32, code = h[0] & 0xff;
        return fail(code == kErrGrid ? APRIL_E_GRID : APRIL_E_INVALID,
                    "polygon " + std::to_string(k) +
                        (code == kErrGrid ? " reaches the outer cell ring or leaves the grid"
                                          : " has a non-lattice coordinate or < 3 distinct vertices"));
    }
    if (h[1] >= (1ull << 32)) {   // (few calls: then the cells themselves are counted)
        BG_TRY(hipMemsetAsync(d_small + 1, 0, 8, s));
        k_count_cells<<<uint32_t(st->cus) * 8, 256, 0, s>>>(d_xy, d_voff, n, nv, g, wide, d_small + 1);
        BG_TRY(hipGetLastError());
        BG_TRY(hipMemcpyAsync(h, d_small, 16, hipMemcpyDeviceToHost, s));
        BG_TRY(hipStreamSynchronize(s));
        if (h[1] >= (1ull << 32))
            return fail(APRIL_E_NOMEM, "more than 2^32 boundary-cell entries in one call: split the collection");
    }

    // polygons of many blocks: items only where they are needed, if that pays
    RowArgs ra{};
    ra.xy = d_xy;
    ra.voff = d_voff;
    ra.box = d_box;
    ra.blocks = d_blocks;
    ra.many = d_many;
    ra.taken = d_taken;
    ra.n_many = h[6] >= kManyTotal ? uint32_t(h[5]) : 0u;
    ra.g = g;
    ra.base = d_base;
    const dim3 row_grid(std::min(ra.n_many, 1024u), kRowBlocks);
    if (ra.n_many) {
        BG_TRY(hipMemsetAsync(d_taken, 0, 4ull * ra.n_many, s));
        k_block_rows<false><<<row_grid, kBlock, 0, s>>>(ra);
        k_many_items<<<blocks_for(ra.n_many), kThreads, 0, s>>>(d_many, d_taken, ra.n_many, d_items);
        BG_TRY(hipGetLastError());
        BG_TRY(hipcub::DeviceScan::ExclusiveSum(d_scan, scan_bytes, d_items, d_base, n + 1, s));
        BG_TRY(hipMemcpyAsync(&items, d_base + n, 8, hipMemcpyDeviceToHost, s));
        BG_TRY(hipStreamSynchronize(s));
    }

    // groups of polygons, one where they have few enough items
    std::vector<uint64_t> base{0, items}, first{0, n};
    if (items > kGroupItems) {
        std::vector<uint64_t> all(n + 1);
        BG_TRY(hipMemcpyAsync(all.data(), d_base, 8 * (n + 1), hipMemcpyDeviceToHost, s));
        BG_TRY(hipStreamSynchronize(s));
        base.assign(1, 0);
        first.assign(1, 0);
        for (uint64_t k = 1; k <= n; k++)
            if (k == n || all[k + 1] - base.back() > kGroupItems) {
                base.push_back(all[k]);
                first.push_back(k);
            }
    }
    uint64_t most = 0, most_polys = 0;
    for (size_t q = 0; q + 1 < base.size(); q++) {
        most = std::max(most, base[q + 1] - base[q]);
        most_polys = std::max(most_polys, first[q + 1] - first[q]);
    }
    int kbits = 2 * g.border;
    while (kbits < 64 && (1ull << (kbits - 2 * g.border)) < most_polys) kbits++;
    size_t sort_bytes = 0, scan2_bytes = 0;
    BG_TRY(hipcub::DeviceRadixSort::SortKeys(nullptr, sort_bytes, (uint64_t *)nullptr, (uint64_t *)nullptr, most, 0,
                                             std::max(kbits, 1), s));
    BG_TRY(hipcub::DeviceScan::ExclusiveSum(nullptr, scan2_bytes, (uint64_t *)nullptr, (uint64_t *)nullptr, most + 1, s));
    const size_t tmp_bytes = std::max(sort_bytes, scan2_bytes);
    if (!sc.reserve(4 * pad(8 * (most + 1)) + 2 * pad(4 * most) + pad(tmp_bytes))) return fail(APRIL_E_NOMEM, "build scratch");
    // the unsorted keys and the starts share an array each with the scans' results
    uint64_t *d_key = sc.get<uint64_t>(most + 1), *d_k0 = sc.get<uint64_t>(most + 1);
    uint64_t *d_na = d_k0, *d_ai = sc.get<uint64_t>(most + 1), *d_nf = sc.get<uint64_t>(most + 1), *d_fi = d_nf;
    uint32_t *d_info = sc.get<uint32_t>(most), *d_place = sc.get<uint32_t>(most);
    void *d_tmp = sc.get<char>(tmp_bytes);
    ItemArgs ia{};
    ia.xy = d_xy;
    ia.voff = d_voff;
    ia.box = d_box;
    ia.blocks = d_blocks;
    ia.base = d_base;
    ia.info = d_info;
    ia.place = d_place;
    ia.many = ra.n_many ? kManyBlocks : ~0u;
    ia.g = g;
    ia.n = n;
    ia.ai = d_ai;
    ia.fi = d_fi;
    // 3-4 and the scans of 5 for one group
    auto count_group = [&](size_t q) -> int {
        ia.first_poly = first[q];
        ia.n_polys = first[q + 1] - first[q];
        ia.item0 = base[q];
        ia.n_items = base[q + 1] - base[q];
        ia.key = d_k0;
        k_item_keys<<<blocks_for(ia.n_items), kThreads, 0, s>>>(ia);
        BG_TRY(hipGetLastError());
        if (ra.n_many) {
            ra.first_poly = ia.first_poly;
            ra.n_polys = ia.n_polys;
            ra.item0 = ia.item0;
            ra.key = d_k0;
            BG_TRY(hipMemsetAsync(d_taken, 0, 4ull * ra.n_many, s));
            k_block_rows<true><<<row_grid, kBlock, 0, s>>>(ra);
            BG_TRY(hipGetLastError());
        }
        BG_TRY(hipcub::DeviceRadixSort::SortKeys(d_tmp, sort_bytes, d_k0, d_key, ia.n_items, 0, std::max(kbits, 1), s));
        ia.key = d_key;
        const uint32_t nb = uint32_t(std::min<uint64_t>((ia.n_items + 3) / 4, uint64_t(st->cus) * 64));
        k_item_places<<<blocks_for(ia.n_items), kThreads, 0, s>>>(ia);
        if (wide) k_items<Wide, false><<<nb, kBlock, 0, s>>>(ia);
        else k_items<Narrow, false><<<nb, kBlock, 0, s>>>(ia);
        k_item_starts<<<blocks_for(ia.n_items + 1), kThreads, 0, s>>>(ia, d_na, d_nf);
        BG_TRY(hipGetLastError());
        BG_TRY(hipcub::DeviceScan::ExclusiveSum(d_tmp, scan2_bytes, d_na, d_ai, ia.n_items + 1, s));
        BG_TRY(hipcub::DeviceScan::ExclusiveSum(d_tmp, scan2_bytes, d_nf, d_fi, ia.n_items + 1, s));
        return APRIL_OK;
    };
    const size_t groups = base.size() - 1;
    std::vector<uint64_t> ga(groups + 1, 0), gf(groups + 1, 0);   // intervals before each group
    for (size_t q = 0; q < groups; q++) {
        if (int rc = count_group(q)) return rc;
        uint64_t tot[2] = {0, 0};
        BG_TRY(hipMemcpyAsync(&tot[0], d_ai + ia.n_items, 8, hipMemcpyDeviceToHost, s));
        BG_TRY(hipMemcpyAsync(&tot[1], d_fi + ia.n_items, 8, hipMemcpyDeviceToHost, s));
        BG_TRY(hipStreamSynchronize(s));
        ga[q + 1] = ga[q] + tot[0];
        gf[q + 1] = gf[q] + tot[1];
    }
    const uint64_t n_a = ga[groups], n_f = gf[groups];

    // the lists, in the layout april_lists_to_device gives raw lists
    auto *L = new (std::nothrow) april_lists;
    if (!L) return fail(APRIL_E_NOMEM, "out of host memory");
    auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
    const size_t b_off = up(8 * (n + 1)), b_a = up(4 * std::max<uint64_t>(n_a, 1)), b_f = up(4 * std::max<uint64_t>(n_f, 1));
    const size_t total = 2 * b_off + 2 * b_a + 2 * b_f;
    hipError_t e = hipMalloc(&L->d.block, total);
    if (e != hipSuccess) {
        delete L;
        return fail(APRIL_E_NOMEM, std::string("hipMalloc lists: ") + hipGetErrorString(e));
    }
    char *p = static_cast<char *>(L->d.block);
    L->d.off_a = reinterpret_cast<uint64_t *>(p); p += b_off;
    L->d.off_f = reinterpret_cast<uint64_t *>(p); p += b_off;
    L->d.start_a = reinterpret_cast<uint32_t *>(p); p += b_a;
    L->d.end_a = reinterpret_cast<uint32_t *>(p); p += b_a;
    L->d.start_f = reinterpret_cast<uint32_t *>(p); p += b_f;
    L->d.end_f = reinterpret_cast<uint32_t *>(p);
    L->d.bytes = total;
    unsigned int *d_bad_slot = reinterpret_cast<unsigned int *>(d_small + 2);   // then: longest list, long A-lists
    ia.off_a = L->d.off_a;
    ia.off_f = L->d.off_f;
    ia.sa = L->d.start_a;
    ia.ea = L->d.end_a;
    ia.sf = L->d.start_f;
    ia.ef = L->d.end_f;
    ia.n_a = n_a;
    ia.n_f = n_f;
    ia.bad_slot = d_bad_slot;
    for (size_t q = 0; q < groups && e == hipSuccess; q++) {
        if (groups > 1 && count_group(q)) {   // (one group: its arrays are still there)
            e = hipErrorUnknown;
            break;
        }
        ia.a0 = ga[q];
        ia.f0 = gf[q];
        const uint32_t nb = uint32_t(std::min<uint64_t>((ia.n_items + 3) / 4, uint64_t(st->cus) * 64));
        if (wide) k_items<Wide, true><<<nb, kBlock, 0, s>>>(ia);
        else k_items<Narrow, true><<<nb, kBlock, 0, s>>>(ia);
        e = hipGetLastError();
    }
    if (e == hipSuccess && launch_list_stats(L->d.off_a, L->d.off_f, n, d_small + 3, s)) e = hipErrorUnknown;
    uint64_t last[3] = {0, 0, 0};   // bad_slot, longest list, A-lists that need a coarse table
    if (e == hipSuccess) e = hipMemcpyAsync(last, d_bad_slot, 24, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);   // the scratch is released after this call
    if (e != hipSuccess || last[0]) {
        (void)hipFree(L->d.block);
        delete L;
        return e != hipSuccess ? fail(APRIL_E_HIP, std::string("build: ") + hipGetErrorString(e))
                               : fail(APRIL_E_CORRUPT, "build: inconsistent interval ends");
    }
    L->grid = *grid;
    L->partition_key = 0;
    L->n = n;
    L->n_a = n_a;
    L->n_f = n_f;
    L->device = dev;
    L->codec = APRIL_CODEC_RAW;
    L->sound = true;
    L->max_len = uint32_t(std::min<uint64_t>(last[1], 0xfffffffeull));
    if (int rc = summaries ? launch_summaries(L, last[2], L->d.start_a, L->d.end_a, L->d.start_f, L->d.end_f, s)
                           : APRIL_OK) {
        april_lists_free(L);
        return rc;
    }
    if (e = hipStreamSynchronize(s); e != hipSuccess) {   // complete on return, for any stream
        april_lists_free(L);
        return fail(APRIL_E_HIP, std::string("build: ") + hipGetErrorString(e));
    }
    *out = L;
    return APRIL_OK;
}
