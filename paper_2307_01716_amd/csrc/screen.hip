// Screening: most candidate pairs are decided from a summary of each object,
// before any of the join kernels reads the object's lists.
//
// Every object of a device collection has a summary of 64 intervals, one per
// lane of a wavefront, made once when the lists are uploaded or built:
//   TF, lanes 0..31   its 32 longest F-intervals, each inside an A-interval;
//   H, lanes 32..63   its hull: the A-list with all but its 31 widest gaps
//                     closed, so every A-interval lies in one of 32.
// (Lists are sorted and disjoint and F lies inside A: those that were not
// validated are checked at upload, and have no summaries where it is otherwise.)
// Against the A-list of the other object, X, these give two one-sided tests:
//   - a TF interval that overlaps A(X): that is an AF overlap, and, as it lies
//     in an A-interval, an AA overlap too: Alg. 2 answers true hit;
//   - no H interval overlaps A(X): no A-interval does: true negative.
// Anything else is left to the join kernels.  X's A-list is held in LDS; for an
// A-list of kExact intervals or more a coarse table of X stands in for it: its
// 127 longest A-intervals in the first test (a subset: an overlap with one is
// an overlap with A(X)), its hull of 127 in the second (a superset).  A wave
// keeps X while consecutive pairs share their R object; one search of the table
// by all lanes makes both tests of a pair.  Where the other object has a
// coarse table too, a pair that is still open is tested once more with that
// table's 127 longest F-intervals and its hull of 127.
//
// The two tests decide 95% of the at-scale join's pairs (98% of its true hits,
// 92% of its true negatives) and 93% of a partition's, whose lists are
// fourteen times as long.  32 + 32 intervals, because a summary then is one
// coalesced 512-byte load and a pair one search; 16 + 16 leave twice as many
// pairs to the joins, each of which costs several times a screened pair.
//
// Measured on one MI355X, whole calls without screening and now, with the open
// pairs listed for k_open: at scale (200k x 200k, 4.5M pairs) 1.96 and 0.64 ms,
// of which this kernel 0.40; the plain schedule at 100k x 100k 1.50 and 0.32 ms;
// a partition of 10k x 10k objects of 2,250 A-intervals 2.51 and 0.37 ms raw,
// 8k x 8k 3.37 and 0.53 ms compressed; 40k x 40k with 300 complex objects a side
// 1.99 and 0.45 ms; 100k x 100k within joins 0.95 and 0.43 ms, linestrings 0.93
// and 0.30.  Making the summaries takes 0.7 ms for 200k objects.  The kernel issues 38
// vector instructions per pair, at 0.63 to 0.68 of the issue peak; two pairs'
// searches side by side gained nothing at scale (0.42 ms).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "internal.hpp"

namespace april {
namespace {

constexpr uint32_t kSumHalf = kSumEntries / 2;    // TF intervals; hull intervals
// longest list that a single wave summarizes; longer ones get 16 waves (a list
// is read twice per selection, and the skewed workload has lists of 200,000)
constexpr uint32_t kOneWave = 2048;

struct SumBuild {
    ListView A, F;
    uint64_t n;
    uint64_t *sum;
    uint32_t *slot, *coarse, *taken;   // taken[0]: coarse tables given out; taken[1]: objects queued
    uint32_t *queue;                   // objects with a longer list than kOneWave
    uint32_t tables, queue_cap;
    uint32_t sample;                   // no F-lists: TF are 32 of the A-list, evenly spaced (linestrings)
    uint32_t by_slot, min_len;         // compressed lists: objects of min_len A-intervals or more have a summary,
                                       // numbered like their coarse tables
};

// Value bins for the selection of the largest: the position of the leading
// bit and the three bits below it, so a bin spans 12.5%.
__device__ __forceinline__ uint32_t bin_of(uint32_t v) {
    v = max(v, 1u);
    const uint32_t b = 31u - uint32_t(__builtin_clz(v));
    return b * 8 + (b >= 3 ? (v >> (b - 3)) & 7u : (v << (3 - b)) & 7u);
}

template <int W>
__device__ __forceinline__ void group_sync() {
    if (W == 1) wave_lds_sync();
    else __syncthreads();
}

// Selection of the K largest of m values by bins: every value in a bin above
// `tie`, and the first `take` (by position) of those in it.
struct Cut {
    uint32_t tie, take;
};

__device__ __forceinline__ Cut find_cut(const uint32_t *hist, uint32_t K, uint32_t lane) {
    // lane l holds bins 255 - 4l ... 252 - 4l
    uint32_t c[4], s = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) s += c[i] = hist[255 - 4 * lane - i];
    uint32_t before = s;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(before, d);
        if (lane >= uint32_t(d)) before += o;
    }
    before -= s;
    uint32_t tie = 0, take = 0;
    bool mine = false;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (!mine && before <= K && before + c[i] > K) {
            mine = true;
            tie = 255 - 4 * lane - i;
            take = K - before;
        }
        before += c[i];
    }
    const uint64_t at = __ballot(mine);
    if (!at) return Cut{0, 0xffffffffu};   // at most K values: all of them
    const int l = int(__builtin_ctzll(at));
    return Cut{uniform(__shfl(tie, l)), uniform(__shfl(take, l))};
}

// The histogram of value(0 .. m).
template <int W, class V>
__device__ __forceinline__ void histogram(uint32_t *hist, uint32_t m, V value, uint32_t tid) {
    group_sync<W>();
    for (uint32_t i = tid; i < 256; i += 64 * W) hist[i] = 0;
    group_sync<W>();
    for (uint32_t j = tid; j < m; j += 64 * W) atomicAdd(&hist[bin_of(value(j))], 1u);
    group_sync<W>();
}

// put(rank, j) for every selected j, ranks in the order of positions.  Wave w
// takes a contiguous share of the positions.
template <int W, class V, class P>
__device__ __forceinline__ void select(Cut cut, uint32_t m, V value, P put, uint32_t (*part)[2], uint32_t w,
                                       uint32_t lane) {
    const uint32_t share = W == 1 ? m : ((m + W - 1) / W + 63) / 64 * 64;
    const uint32_t j0 = min(m, w * share), j1 = min(m, j0 + share);
    uint32_t above = 0, ties = 0;   // selected, tied, in the positions before
    if (W > 1) {
        uint32_t a = 0, t = 0;
        for (uint32_t j = j0; j < j1; j += 64) {
            const uint32_t b = j + lane < j1 ? bin_of(value(j + lane)) : 0u;
            a += uint32_t(__popcll(__ballot(j + lane < j1 && b > cut.tie)));
            t += uint32_t(__popcll(__ballot(j + lane < j1 && b == cut.tie)));
        }
        __syncthreads();
        if (lane == 0) {
            part[w][0] = a;
            part[w][1] = t;
        }
        __syncthreads();
        for (uint32_t k = 0; k < w; k++) {
            above += part[k][0];
            ties += part[k][1];
        }
    }
    uint32_t rank = above + min(ties, cut.take);
    const uint64_t below = (1ull << lane) - 1;
    for (uint32_t j = j0; j < j1; j += 64) {
        const bool in = j + lane < j1;
        const uint32_t b = in ? bin_of(value(j + lane)) : 0u;
        const bool tied = in && b == cut.tie;
        const uint64_t mt = __ballot(tied);
        const bool sel = in && (b > cut.tie || (tied && ties + uint32_t(__popcll(mt & below)) < cut.take));
        const uint64_t ms = __ballot(sel);
        if (sel) put(rank + uint32_t(__popcll(ms & below)), j + lane);
        ties += uint32_t(__popcll(mt));
        rank += uint32_t(__popcll(ms));
    }
}

struct SumLds {
    uint32_t hist[256];
    uint32_t sum[2 * kSumEntries];   // (start, end) pairs
    uint32_t coarse[kTable];
    uint32_t part[16][2];
};

// The hull of X.A with K gaps kept: hull interval i ends at the i-th kept gap
// and the next one starts behind it.  end/start: its arrays, `step` words
// apart.
template <int W>
__device__ __forceinline__ void hull(const uint32_t *as, const uint32_t *ae, uint32_t na, Cut cut, uint32_t K,
                                     uint32_t *start, uint32_t *end, uint32_t step, SumLds &l, uint32_t w,
                                     uint32_t lane) {
    auto gap = [&](uint32_t j) { return as[j + 1] - ae[j]; };
    if (na == 0) return;
    if (w == 0 && lane == 0) {
        start[0] = as[0];
        end[min(K, na - 1) * step] = ae[na - 1];
    }
    select<W>(cut, na - 1, gap, [&](uint32_t i, uint32_t j) {
        end[i * step] = ae[j];
        start[(i + 1) * step] = as[j + 1];
    }, l.part, w, lane);
}

// One object's summary, and its coarse table when `slot` is given.  Entries
// not used are empty on the summary's side (end 0) and beyond every key on the
// table's (0xFFFFFFFF), as in the joins' LDS tiles.
template <int W>
__device__ void summarize(const SumBuild &b, uint64_t k, uint32_t slot, SumLds &l, uint32_t w, uint32_t lane) {
    const uint32_t tid = w * 64 + lane;
    const uint64_t a0 = b.A.off[k], f0 = b.sample ? 0 : b.F.off[k];
    const uint32_t na = uint32_t(b.A.off[k + 1] - a0), nf = b.sample ? 0u : uint32_t(b.F.off[k + 1] - f0);
    const uint32_t *as = b.A.s + a0, *ae = b.A.e + a0, *fs = b.F.s + f0, *fe = b.F.e + f0;
    group_sync<W>();
    for (uint32_t i = tid; i < 2 * kSumEntries; i += 64 * W) l.sum[i] = (i & 1) ? 0u : 0xffffffffu;
    if (slot != kNoSlot)
        for (uint32_t i = tid; i < kTable; i += 64 * W) l.coarse[i] = 0xffffffffu;
    if (b.sample) {
        if (tid < min(na, kSumHalf)) {
            const uint32_t j = na <= kSumHalf ? tid : uint32_t(uint64_t(na - 1) * tid / (kSumHalf - 1));
            l.sum[2 * tid] = as[j];
            l.sum[2 * tid + 1] = ae[j];
        }
    } else {
    // TF
    auto flen = [&](uint32_t j) { return fe[j] - fs[j]; };
    histogram<W>(l.hist, nf, flen, tid);
    select<W>(find_cut(l.hist, kSumHalf, lane), nf, flen, [&](uint32_t i, uint32_t j) {
        l.sum[2 * i] = fs[j];
        l.sum[2 * i + 1] = fe[j];
    }, l.part, w, lane);
    if (slot != kNoSlot)
        select<W>(find_cut(l.hist, kCoarse - 1, lane), nf, flen, [&](uint32_t i, uint32_t j) {
            l.coarse[4 * kCoarse + i] = fe[j];
            l.coarse[5 * kCoarse + i] = fs[j];
        }, l.part, w, lane);
    }
    // H, and the coarse hull from the same histogram
    auto gap = [&](uint32_t j) { return as[j + 1] - ae[j]; };
    const uint32_t ng = na ? na - 1 : 0u;
    histogram<W>(l.hist, ng, gap, tid);
    hull<W>(as, ae, na, find_cut(l.hist, kSumHalf - 1, lane), kSumHalf - 1, l.sum + kSumEntries,
            l.sum + kSumEntries + 1, 2, l, w, lane);
    if (slot != kNoSlot) {
        hull<W>(as, ae, na, find_cut(l.hist, kCoarse - 2, lane), kCoarse - 2, l.coarse + 3 * kCoarse,
                l.coarse + kCoarse, 1, l, w, lane);
        auto alen = [&](uint32_t j) { return ae[j] - as[j]; };
        histogram<W>(l.hist, na, alen, tid);
        select<W>(find_cut(l.hist, kCoarse - 1, lane), na, alen, [&](uint32_t i, uint32_t j) {
            l.coarse[i] = ae[j];
            l.coarse[2 * kCoarse + i] = as[j];
        }, l.part, w, lane);
    }
    group_sync<W>();
    if (w == 0) {
        const uint64_t at = b.by_slot ? slot : k;
        b.sum[at * kSumEntries + lane] = (uint64_t(l.sum[2 * lane + 1]) << 32) | l.sum[2 * lane];
    }
    if (slot != kNoSlot)
        for (uint32_t i = tid; i < kTable; i += 64 * W) b.coarse[uint64_t(slot) * kTable + i] = l.coarse[i];
}

// Objects whose lists one wave summarizes; the others are queued.  Numbers
// the coarse tables (in no particular order).
__global__ __launch_bounds__(kBlock) void k_summaries(SumBuild b) {
    __shared__ SumLds lds[kWavesPerBlock];
    const uint32_t lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    const uint64_t waves = uint64_t(gridDim.x) * kWavesPerBlock;
    for (uint64_t k = uint64_t(blockIdx.x) * kWavesPerBlock + w; k < b.n; k += waves) {
        const uint32_t na = uint32_t(b.A.off[k + 1] - b.A.off[k]);
        const uint32_t nf = b.sample ? 0u : uint32_t(b.F.off[k + 1] - b.F.off[k]);
        uint32_t slot = kNoSlot;
        if (b.tables && na >= (b.by_slot ? b.min_len : kExact)) {
            if (lane == 0) slot = atomicAdd(&b.taken[0], 1u);
            slot = uniform(__shfl(slot, 0));
            if (slot >= b.tables) slot = kNoSlot;
        }
        if (lane == 0) b.slot[k] = slot;
        if (b.by_slot && slot == kNoSlot) continue;
        if (max(na, nf) > kOneWave) {
            if (lane == 0) {
                const uint32_t q = atomicAdd(&b.taken[1], 1u);
                if (q < b.queue_cap) b.queue[q] = uint32_t(k);
            }
            continue;
        }
        summarize<1>(b, k, slot, lds[w], 0, lane);
    }
}

__global__ __launch_bounds__(1024) void k_summaries_long(SumBuild b) {
    __shared__ SumLds lds;
    const uint32_t lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    const uint32_t n = min(b.taken[1], b.queue_cap);
    for (uint32_t q = blockIdx.x; q < n; q += gridDim.x) {
        const uint32_t k = b.queue[q];
        __syncthreads();
        summarize<16>(b, k, b.slot[k], lds, w, lane);
    }
}

__global__ void k_clear_taken(uint32_t *t) { t[threadIdx.x] = 0; }

// ---------------------------------------------------------------- screening

struct ScreenArgs {
    FilterArgs f;
    const uint64_t *sum;             // S's summaries
    const uint32_t *s_slot;          // their numbers (compressed lists; else the S id)
    const uint32_t *r_slot, *coarse;      // R's coarse tables
    const uint32_t *s_table, *s_coarse;   // and S's
    unsigned int *ctr;
    uint32_t xcds;
    uint32_t take;                   // pairs a wave takes at a time (at most 64)
    uint32_t raw;                    // R's A-lists can be read (not compressed)
    uint32_t give_up;                // see kProbe
    OpenLists open;
};

// LDS place of a table's entry i: a word is left out after every 64.  The
// entries that a round of the search compares lie a power of two apart, which
// without that is the same bank for up to four of them in most rounds
// (1.7 conflict cycles per LDS instruction).
__device__ __forceinline__ constexpr uint32_t padded(uint32_t i) { return i + (i >> 6); }
constexpr uint32_t kStarts = kExact + kExact / 64;   // from an end to its start

// The first entry of a table (P2 entries, the last ones padding) that ends above `key`.
template <int P2>
__device__ __forceinline__ const uint32_t *find(const uint32_t *ends, uint32_t key) {
    const uint32_t *p = ends;
#pragma unroll
    for (uint32_t S = P2 / 2; S > 0; S >>= 1) p = p[padded(S - 1)] <= key ? p + padded(S) : p;
    return p;
}

// (size: a power of two, 0 for a coarse table)
__device__ __forceinline__ const uint32_t *find_any(const uint32_t *ends, uint32_t size, uint32_t key) {
    if (size == 64) return find<64>(ends, key);
    if (size == 128 || size == 0) return find<128>(ends, key);
    if (size == 256) return find<256>(ends, key);
    return find<kExact>(ends, key);
}
static_assert(kCoarse == 128, "find_any");

// Does [s, e) overlap an interval of the table?  (The first one that ends
// above s has to start below e.)
__device__ __forceinline__ bool search_any(const uint32_t *ends, uint32_t size, uint32_t s, uint32_t e) {
    return find_any(ends, size, s)[kStarts] < e;
}

// A table place's entry number (places step over one word in 65).
__device__ __forceinline__ uint32_t entry_at(const uint32_t *ends, const uint32_t *p) {
    const uint32_t q = uint32_t(p - ends);
    return q - ((q * 1009) >> 16);   // q / 65 for q < 520
}

// What is screened for.  Alg. 2; within joins (is r within s?); polygons
// against linestrings, whose runs of cells stand for A-lists and, 32 of them
// evenly spaced, for TF.
//
// Within joins: no H interval of s overlapping A(r) is a true negative as
// before.  A TF interval of s that overlaps A(r) is an overlap of the A-lists;
// if then some A-interval of r lies in no hull interval of s, it lies in no
// F-interval either: indecisive.  (The hull intervals are disjoint, so the
// A-intervals inside them are counted by two searches each.)  Decides 90% of
// the at-scale pairs.
//
// Linestrings: a run that overlaps F(p) is a true hit, no hull interval of the
// runs overlapping A(p) a true negative; 94% of the pairs.  Both lists of the
// polygon are in LDS (or its coarse table's longest F-intervals and hull).
constexpr int kAlg2 = 0, kWithin = 1, kLines = 2;

// One word per active lane from global memory straight into LDS, lane l's at dst[l].
__device__ __forceinline__ void lds_dma(const uint32_t *src, uint32_t *dst) {
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)dst, 4, 0, 0);
}

// A wave takes up to 64 pairs at a time from its XCD's range, a lane reading one
// pair's ids and the bounds of its R list, then goes through them one by one;
// the next pair's summary is loaded before the current one is searched.  Every
// pair costs about the same, so the blocks are dealt out without counters.
//
// Where more than give_up eighths of the pairs that a wave has looked at stayed
// open, it looks at kProbe of its next ones and leaves the others to the joins
// (those with a coarse table aside: such joins take far longer than a look).
// That is the batched calls whose joins are cheap: 500 x 500 adjacent polygons
// with themselves, 2.2M pairs of which 89% are open, 1.55 and now 1.51 ms (1.29
// without screening), within 1.36 and 1.22 (1.08), with the edges as linestrings
// 0.80 and 0.61 (0.50).  The lines lie where the two break even when fewer are
// open: of pairs half of which are decided the linestrings take 0.64 ms at 5 and
// at 8 eighths, 0.67 at 4.
constexpr uint32_t kProbe = 8;

template <int MODE>
__global__ __launch_bounds__(kBlock, MODE == kLines ? 4 : 8) void k_screen(ScreenArgs a) {
    // X: ends, then starts (linestrings: of A, then of F)
    constexpr uint32_t kF = MODE == kLines ? 2 * kStarts : 0;
    __shared__ uint32_t lds[kWavesPerBlock][kF + 2 * kStarts];
    const uint32_t lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    uint32_t *const t = lds[w];
    const uint32_t *const hull = t + padded(kCoarse);               // a coarse table's second list
    const uint32_t *const half = lane < kSumHalf ? t : hull;        // the coarse list a lane searches
    const uint32_t *const whole = MODE == kLines && lane < kSumHalf ? t + kF : t;   // and the exact one
    const uint32_t xcd = blockIdx.x % a.xcds, bx = blockIdx.x / a.xcds, nbx = gridDim.x / a.xcds;
    const uint64_t lo = a.f.n_pairs * xcd / a.xcds, hi = a.f.n_pairs * (xcd + 1) / a.xcds;
    unsigned long long c_tn = 0, c_th = 0, c_ind = 0;
    uint32_t x_lo = 0, x_hi = 0;           // (within joins: its A-list's first start, last end)
    uint32_t cached = kNoSlot, size = 0;   // the R object in t; its table's entries, a power of two (0: coarse)
    bool mostly_open = false;              // the wave's last pairs
    for (uint64_t g0 = lo + uint64_t(a.take) * (bx * kWavesPerBlock + w); g0 < hi;
         g0 += uint64_t(a.take) * nbx * kWavesPerBlock) {
        const uint64_t p = g0 + lane;
        uint32_t r = 0, s_at = 0, nar = 0, slot = kNoSlot, s_tab = kNoSlot;
        uint64_t ar0 = 0, fr0 = 0;
        uint32_t nfr = 0;
        bool todo_me = false, few = false;   // few: neither object has a coarse table
        uint32_t vv = APRIL_BAD_PAIR;
        const bool mine = lane < a.take && p < hi;
        if (mine) {
            r = a.f.r[p];
            const uint32_t s = a.f.s[p];
            if ((r < a.f.n_r) & (s < a.f.n_s)) {
                vv = kPending;
                ar0 = a.f.Ar.off[r];
                nar = uint32_t(a.f.Ar.off[r + 1] - ar0);
                if (MODE == kLines) {
                    fr0 = a.f.Fr.off[r];
                    nfr = uint32_t(a.f.Fr.off[r + 1] - fr0);
                } else {
                    s_tab = a.s_table[s];
                }
                s_at = a.s_slot ? s_tab : s;
                const bool exact = a.raw && max(nar, nfr) < kExact;
                if (!exact) slot = a.r_slot[r];
                todo_me = s_at != kNoSlot && (exact || slot != kNoSlot);
                few = slot == kNoSlot && s_tab == kNoSlot;
                todo_me &= !(few && mostly_open && lane >= kProbe);
            }
        }
        // pair k's R object into LDS, unless it is there
        auto load_x = [&](uint32_t k) {
            const uint32_t key = __builtin_amdgcn_readlane(r, k);
            if (key == cached) return;
            cached = key;
            const uint32_t sl = __builtin_amdgcn_readlane(slot, k);
            wave_lds_sync();
            if (sl == kNoSlot) {
                const uint32_t n = __builtin_amdgcn_readlane(nar, k);
                const uint32_t nf = MODE == kLines ? __builtin_amdgcn_readlane(nfr, k) : 0u, nm = max(n, nf);
                auto copy = [&](const uint32_t *xs, const uint32_t *xe, uint32_t m, uint32_t *to) {
#pragma unroll 1
                    for (uint32_t i = 0; i < size; i += 64) {
                        if (i + lane < m) {
                            lds_dma(xe + i + lane, to + padded(i));
                            lds_dma(xs + i + lane, to + kStarts + padded(i));
                        } else {
                            to[padded(i) + lane] = 0xffffffffu;
                            to[kStarts + padded(i) + lane] = 0xffffffffu;
                        }
                    }
                };
                auto lane64 = [&](uint64_t v) {
                    return (uint64_t(uint32_t(__builtin_amdgcn_readlane(uint32_t(v >> 32), k))) << 32) |
                           uint32_t(__builtin_amdgcn_readlane(uint32_t(v), k));
                };
                size = nm < 64 ? 64u : nm < 128 ? 128u : nm < 256 ? 256u : kExact;   // above nm: a padding entry
                const uint64_t at = lane64(ar0);
                copy(a.f.Ar.s + at, a.f.Ar.e + at, n, t);
                if (MODE == kLines) {
                    const uint64_t ft = lane64(fr0);
                    copy(a.f.Fr.s + ft, a.f.Fr.e + ft, nf, t + kF);
                }
            } else {
                // (linestrings: the longest F-intervals in the place of the longest A-intervals)
                const uint32_t *c = a.coarse + uint64_t(sl) * kTable, *first = c + (MODE == kLines ? 4 * kCoarse : 0);
                const uint32_t to_start = MODE == kLines ? kCoarse : 2 * kCoarse;
                size = 0;
#pragma unroll
                for (uint32_t i = 0; i < kCoarse; i += 64) {
                    lds_dma(first + i + lane, t + padded(i));
                    lds_dma(first + to_start + i + lane, t + kStarts + padded(i));
                    lds_dma(c + kCoarse + i + lane, t + padded(kCoarse + i));
                    lds_dma(c + 3 * kCoarse + i + lane, t + kStarts + padded(kCoarse + i));
                }
            }
            __builtin_amdgcn_s_waitcnt(0);   // the copies, all under way at once, have landed
            wave_lds_sync();
            if (MODE == kWithin) {
                const uint32_t n = size ? __builtin_amdgcn_readlane(nar, k) : kCoarse - 1;
                const uint32_t at = size ? 0u : kCoarse;   // a coarse table's hull has the list's ends
                x_lo = uniform(t[padded(at) + kStarts]);
                x_hi = n ? uniform(t[padded(at + n - 1)]) : 0u;
            }
        };
        uint64_t todo = __ballot(todo_me);
        uint32_t kn = todo ? uint32_t(__builtin_ctzll(todo)) : 0u;
        uint64_t y_next = 0;
        if (todo) y_next = a.sum[uint64_t(__builtin_amdgcn_readlane(s_at, kn)) * kSumEntries + lane];
        while (todo) {
            const uint32_t k = kn;
            const uint64_t y = y_next;
            todo &= todo - 1;
            if (todo) {
                kn = uint32_t(__builtin_ctzll(todo));
                y_next = a.sum[uint64_t(__builtin_amdgcn_readlane(s_at, kn)) * kSumEntries + lane];
            }
            load_x(k);
            const uint32_t ys = uint32_t(y), ye = uint32_t(y >> 32);
            const uint64_t m = __ballot(search_any(size ? whole : half, size, ys, ye));
            uint32_t v;
            if (MODE == kWithin) {
                v = uint32_t(m >> 32) ? kPending : APRIL_TN;
                const uint64_t some = __ballot(ye != 0);
                if (uint32_t(m) && v == kPending &&
                    (x_lo < uint32_t(__builtin_amdgcn_readlane(ys, kSumHalf)) ||
                     x_hi > uint32_t(__builtin_amdgcn_readlane(ye, 63 - __builtin_clzll(some))))) {
                    v = APRIL_INDECISIVE;   // beyond the hull at one end
                } else if (uint32_t(m) && v == kPending) {
                    // the A-intervals (of a coarse table: its longest) inside each hull interval
                    const uint32_t *p0 = find_any(t, size, ys), *p1 = find_any(t, size, ye);
                    const uint32_t i0 = entry_at(t, p0) + (p0[kStarts] < ys ? 1u : 0u), i1 = entry_at(t, p1);
                    uint32_t in = lane >= kSumHalf && ye != 0 && i1 > i0 ? i1 - i0 : 0u;
                    for (int off = 32; off > 0; off >>= 1) in += __shfl_xor(in, off);
                    const uint32_t n = size ? __builtin_amdgcn_readlane(nar, k) : kCoarse - 1;
                    if (in < n) v = APRIL_INDECISIVE;
                }
            } else {
                v = uint32_t(m) ? APRIL_TH : uint32_t(m >> 32) ? kPending : APRIL_TN;
            }
            vv = lane == k ? v : vv;
        }
        {
            const uint64_t looked = __ballot(todo_me && few), left = __ballot(todo_me && few && vv == kPending);
            mostly_open = 8 * uint32_t(__popcll(left)) > a.give_up * uint32_t(__popcll(looked));
        }
        // once more, with S's coarse table where it has one (padding entries
        // overlap nothing); apart from the loop above, which it would slow down
        todo = MODE == kAlg2 ? __ballot(todo_me && vv == kPending && s_tab != kNoSlot) : 0;
        while (todo) {
            const uint32_t k = uint32_t(__builtin_ctzll(todo));
            todo &= todo - 1;
            const uint32_t *c = a.s_coarse + uint64_t(__builtin_amdgcn_readlane(s_tab, k)) * kTable;
            uint32_t fs[2], fe[2], hs[2], he[2];
#pragma unroll
            for (uint32_t i = 0; i < 2; i++) {
                fe[i] = c[4 * kCoarse + 64 * i + lane];
                fs[i] = c[5 * kCoarse + 64 * i + lane];
                he[i] = c[kCoarse + 64 * i + lane];
                hs[i] = c[3 * kCoarse + 64 * i + lane];
            }
            load_x(k);
            bool f = false, h = false;
#pragma unroll
            for (uint32_t i = 0; i < 2; i++) {
                f |= search_any(t, size, fs[i], fe[i]);
                h |= search_any(size ? t : hull, size, hs[i], he[i]);
            }
            const uint32_t v = __any(f) ? APRIL_TH : __any(h) ? kPending : APRIL_TN;
            vv = lane == k ? v : vv;
        }
        if (a.open.pairs) {
            const bool open = mine && vv == kPending, big = slot != kNoSlot || s_tab != kNoSlot;
            uint32_t *const list = a.open.pairs + uint64_t(xcd) * (a.open.cap + a.open.long_cap);
            const uint64_t few = __ballot(open && !big), lng = __ballot(open && big);
            uint32_t at = 0;   // lane 0: of the others, lane 1: of the long ones
            if (lane < 2 && (lane ? lng : few))
                at = atomicAdd(&(lane ? a.open.long_fill : a.open.fill)[xcd * kCtrStride],
                               uint32_t(__popcll(lane ? lng : few)));
            const uint32_t at_few = __shfl(at, 0), at_lng = __shfl(at, 1);
            at = (big ? at_lng : at_few) + uint32_t(__popcll((big ? lng : few) & ((1ull << lane) - 1)));
            if (open && at < (big ? a.open.long_cap : a.open.cap)) {
                list[(big ? a.open.cap : 0u) + at] = uint32_t(p);
                vv = kListed;
            }
        }
        if (mine) {
            a.f.verdict[p] = uint8_t(vv);
            c_tn += vv == APRIL_TN;
            c_th += vv == APRIL_TH;
            if (MODE == kWithin) c_ind += vv == APRIL_INDECISIVE;
        }
    }
    if (a.f.counts) {
        for (int off = 32; off > 0; off >>= 1) {
            c_tn += __shfl_down(c_tn, off);
            c_th += __shfl_down(c_th, off);
            if (MODE == kWithin) c_ind += __shfl_down(c_ind, off);
        }
        const unsigned long long v[3] = {c_tn, c_th, c_ind};
        if (lane == 0) add_totals(a.ctr, blockIdx.x * kWavesPerBlock + w, v, 3);
    }
}

// A wave per object: are its lists sorted, disjoint, of no empty interval, and
// its F-intervals inside A-intervals?
__global__ __launch_bounds__(kBlock) void k_check_lists(ListView A, ListView F, uint64_t n, unsigned int *bad) {
    const uint32_t lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    const uint64_t waves = uint64_t(gridDim.x) * kWavesPerBlock;
    bool wrong = false;
    for (uint64_t k = uint64_t(blockIdx.x) * kWavesPerBlock + w; k < n; k += waves) {
        const uint64_t a0 = A.off[k], a1 = A.off[k + 1], f1 = F.off[k + 1];
        auto check = [&](const ListView &L, uint64_t t, uint64_t end) {
            wrong |= L.s[t] >= L.e[t] || (t + 1 < end && L.e[t] > L.s[t + 1]);
        };
        for (uint64_t t = a0 + lane; t < a1; t += 64) check(A, t, a1);
        for (uint64_t t = F.off[k] + lane; t < f1; t += 64) {
            check(F, t, f1);
            uint64_t lo = a0, hi = a1;   // the first A-interval that ends at or above F's end
            while (lo < hi) {
                const uint64_t mid = (lo + hi) >> 1;
                if (A.e[mid] >= F.e[t]) hi = mid;
                else lo = mid + 1;
            }
            wrong |= lo == a1 || A.s[lo] > F.s[t];
        }
    }
    if (__any(wrong) && lane == 0) atomicOr(bad, 1u);
}

__global__ void k_list_stats(const uint64_t *off_a, const uint64_t *off_f, uint64_t n, unsigned long long *stats) {
    const uint32_t lane = threadIdx.x & 63;
    unsigned long long longest = 0, longer = 0;
    for (uint64_t k = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < n; k += uint64_t(gridDim.x) * blockDim.x) {
        const unsigned long long na = off_a[k + 1] - off_a[k], nf = off_f[k + 1] - off_f[k];
        longest = max(longest, max(na, nf));
        longer += na >= kExact;
    }
    for (int off = 32; off > 0; off >>= 1) {
        longest = max(longest, (unsigned long long)__shfl_down(longest, off));
        longer += __shfl_down(longer, off);
    }
    if (lane == 0) {
        atomicMax(&stats[0], longest);
        if (longer) atomicAdd(&stats[1], longer);
    }
}

}  // namespace

int launch_list_stats(const uint64_t *off_a, const uint64_t *off_f, uint64_t n, unsigned long long *stats,
                      hipStream_t stream) {
    k_list_stats<<<dim3(uint32_t(std::min<uint64_t>((n + 255) / 256, 256))), dim3(256), 0, stream>>>(off_a, off_f, n,
                                                                                                   stats);
    APRIL_HIP_TRY(hipGetLastError());
    return APRIL_OK;
}

int launch_check_lists(uint64_t n, const uint64_t *off_a, const uint32_t *as, const uint32_t *ae, const uint64_t *off_f,
                       const uint32_t *fs, const uint32_t *fe, unsigned int *bad, hipStream_t stream) {
    k_check_lists<<<dim3(uint32_t(std::min<uint64_t>((n + 3) / 4, 4096))), dim3(kBlock), 0, stream>>>(
        {off_a, as, ae}, {off_f, fs, fe}, n, bad);
    APRIL_HIP_TRY(hipGetLastError());
    return APRIL_OK;
}

// Fewest pairs that are screened: in smaller calls each wave has one pair
// anyway, and screening only comes before its join.  Measured, without and with:
// at-scale objects, plain schedule, 4,204 pairs 30 and 34 us, 16,272 pairs 58
// and 40 us; batched, 4,204 pairs 20 and 21 us, 16,272 pairs 33 and 31 us,
// 65,088 pairs 93 and 55 us.  Long lists, whose joins take far longer, are always
// worth it: 486 pairs of objects of 2,250 A-intervals 293 and 134 us raw, 1384
// and 210 us compressed; 2,804 pairs with some complex objects 442 and 131 us.
constexpr uint64_t kScreenMin = 8192;
constexpr uint64_t kLongMean = 512, kLongMost = 4096;

static bool long_lists(const april_lists_t *L) {
    return L->n_a >= kLongMean * L->n || (L->max_len >= kLongMost && L->max_len != 0xffffffffu);
}

bool can_screen(const april_lists_t *R, const april_lists_t *S, uint64_t n_pairs) {
    if (n_pairs < kScreenMin && !long_lists(R) && !long_lists(S)) return false;
    // (compressed lists: where most objects are long enough to have a summary)
    return R->d.sum && S->d.sum && 2 * R->d.n_sums >= R->n && 2 * S->d.n_sums >= S->n;
}

// Batched calls of more than 2^21 pairs between lists of a few intervals (A-lists
// of fewer than 6 on average on both sides): a look at a summary costs more than
// such a join, most of which take a lane each.  8.6M pairs of lists of 3.4 on
// average: batched 1.02 ms without screening and 1.29 with it, within 2.77 and
// 3.62, 2.8M pairs with linestrings 0.72 and 1.05; 5.9 on average: 1.69 and 1.70,
// 2.76 and 2.59, 0.71 and 0.80; 11: 2.39 and 1.45.  Smaller calls go by the lists
// of open pairs, which are dealt out faster: 0.7M pairs of 3.4 0.23 and 0.15 ms.
static bool cheap_joins(uint64_t intervals_r, uint64_t n_r, uint64_t intervals_s, uint64_t n_s, uint64_t n_pairs) {
    return n_pairs > (1ull << 21) && intervals_r < 6 * n_r && intervals_s < 6 * n_s;
}

bool can_screen_batched(const april_lists_t *R, const april_lists_t *S, uint64_t n_pairs) {
    return can_screen(R, S, n_pairs) && !cheap_joins(R->n_a, R->n, S->n_a, S->n, n_pairs);
}

bool can_screen_lines(const april_lists_t *P, const april_cells_t *L, uint64_t n_pairs) {
    return (n_pairs >= kScreenMin || long_lists(P)) && P->d.sum && L->sum &&
           !cheap_joins(P->n_a, P->n, L->n_runs, L->n, n_pairs);
}

template <int MODE>
static int screen(ScreenArgs &a, const april_lists_t *R, int cus, void *counters, hipStream_t stream) {
    a.give_up = a.open.pairs ? (MODE == kLines ? 5 : 6) : 8;
    a.r_slot = R->d.slot;
    a.coarse = R->d.coarse;
    a.raw = R->codec == APRIL_CODEC_RAW;
    a.ctr = static_cast<unsigned int *>(counters);
    a.xcds = uint32_t(xcd_count(cus));
    // 64 pairs at a time, or what gives every wave some: a pair takes half a
    // microsecond and more after another (16,272 pairs with 64 at a time: 93 us
    // a call, so 31)
    const uint64_t most = uint64_t(cus) * (MODE == kLines ? 4 : 8), waves = most * kWavesPerBlock;
    a.take = uint32_t(std::min<uint64_t>(64, std::max<uint64_t>(1, (a.f.n_pairs + waves - 1) / waves)));
    uint64_t blocks = std::min(most, (a.f.n_pairs + a.take * kWavesPerBlock - 1) / (a.take * kWavesPerBlock));
    blocks = (blocks + a.xcds - 1) / a.xcds * a.xcds;
    k_screen<MODE><<<dim3(uint32_t(blocks)), dim3(kBlock), 0, stream>>>(a);
    APRIL_HIP_TRY(hipGetLastError());
    return APRIL_OK;
}

int launch_screen(const april_lists_t *R, const april_lists_t *S, const FilterArgs &f, int cus, void *counters,
                  hipStream_t stream, bool within, const OpenLists &open) {
    ScreenArgs a{};
    a.f = f;
    a.open = open;
    a.sum = S->d.sum;
    a.s_slot = S->codec == APRIL_CODEC_RAW ? nullptr : S->d.slot;
    a.s_table = S->d.slot;
    a.s_coarse = S->d.coarse;
    return within ? screen<kWithin>(a, R, cus, counters, stream) : screen<kAlg2>(a, R, cus, counters, stream);
}

int launch_screen_lines(const april_lists_t *P, const april_cells_t *L, const FilterArgs &f, int cus, void *counters,
                        hipStream_t stream, const OpenLists &open) {
    ScreenArgs a{};
    a.f = f;
    a.open = open;
    a.sum = L->sum;
    return screen<kLines>(a, P, cus, counters, stream);
}

namespace {

// Summaries of n lists on `stream` into an allocation of their own (null when
// there is no memory for it: lists without summaries are joined without
// screening).  `tables`: coarse tables needed.
struct Made {
    void *block;
    uint64_t *sum;
    uint32_t *slot, *coarse;
    uint64_t sums, bytes;
};

int make_summaries(ListView A, ListView F, uint64_t n, uint64_t intervals, uint64_t tables, bool by_slot, bool sample,
                   hipStream_t stream, Made *out) {
    *out = Made{};
    const uint64_t sums = by_slot ? tables : n;
    if (sums == 0 || n >= 0x7fffffffull || tables >= 0x7fffffffull) return APRIL_OK;
    auto up = [](uint64_t v) { return (v + 255) & ~uint64_t(255); };
    const uint64_t queue = std::min<uint64_t>(n, intervals / kOneWave + 1);
    const uint64_t b_sum = up(8 * kSumEntries * sums), b_coarse = up(4 * kTable * tables), b_slot = up(4 * n);
    const uint64_t total = b_sum + b_coarse + b_slot + up(4 * queue) + 256;
    void *block = nullptr;
    if (hipMalloc(&block, total) != hipSuccess) {
        (void)hipGetLastError();
        return APRIL_OK;
    }
    char *p = static_cast<char *>(block);
    SumBuild b;
    b.A = A;
    b.F = F;
    b.n = n;
    b.sum = reinterpret_cast<uint64_t *>(p); p += b_sum;
    b.coarse = reinterpret_cast<uint32_t *>(p); p += b_coarse;
    b.slot = reinterpret_cast<uint32_t *>(p); p += b_slot;
    b.taken = reinterpret_cast<uint32_t *>(p); p += 256;
    b.queue = reinterpret_cast<uint32_t *>(p);
    b.tables = uint32_t(tables);
    b.queue_cap = uint32_t(queue);
    b.sample = sample ? 1 : 0;
    b.by_slot = by_slot ? 1 : 0;
    b.min_len = kVbyteSummaryMin;
    k_clear_taken<<<1, 2, 0, stream>>>(b.taken);
    k_summaries<<<dim3(uint32_t(std::min<uint64_t>((n + 3) / 4, 4096))), dim3(kBlock), 0, stream>>>(b);
    if (intervals > kOneWave)
        k_summaries_long<<<dim3(uint32_t(std::min<uint64_t>(queue, 512))), dim3(1024), 0, stream>>>(b);
    if (const hipError_t e = hipGetLastError(); e != hipSuccess) {
        (void)hipFree(block);
        return fail(APRIL_E_HIP, std::string("summaries: ") + hipGetErrorString(e));
    }
    *out = Made{block, b.sum, b.slot, b.coarse, sums, total};
    return APRIL_OK;
}

}  // namespace

// `longer`: objects whose A-list has kExact intervals or more (compressed
// lists: kVbyteSummaryMin).  as/ae/fs/fe: the raw arrays (of compressed lists:
// decoded copies).
int launch_summaries(april_lists_t *L, uint64_t longer, const uint32_t *as, const uint32_t *ae, const uint32_t *fs,
                     const uint32_t *fe, hipStream_t stream) {
    Made m;
    if (int rc = make_summaries({L->d.off_a, as, ae}, {L->d.off_f, fs, fe}, L->n, L->n_a + L->n_f, longer,
                                L->codec != APRIL_CODEC_RAW, false, stream, &m))
        return rc;
    L->d.sum_block = m.block;
    L->d.sum = m.sum;
    L->d.slot = m.slot;
    L->d.coarse = m.coarse;
    L->d.n_sums = m.sums;
    L->d.bytes += m.bytes;
    return APRIL_OK;
}

int launch_line_summaries(april_cells_t *C, hipStream_t stream) {
    Made m;
    const ListView runs{C->d_off, C->d_start, C->d_end};
    if (int rc = make_summaries(runs, runs, C->n, C->n_runs, 0, false, true, stream, &m)) return rc;
    C->sum_block = m.block;
    C->sum = m.sum;
    return APRIL_OK;
}

}  // namespace april
