// MBR filter of the served form (Sec. 4.3.1: a query polygon's MBR selects
// the data polygons whose MBRs intersect it, then the intermediate filter
// runs on those pairs).
//
// S is indexed by a uniform G x G grid over its extent: every S object is
// registered in each grid cell its MBR overlaps (CSR cell -> ids), and its
// integer cell range is stored beside its box.  A query probes the cells its
// MBR overlaps and reports (q, s) only from the cell holding the lower-left
// corner of the two MBRs' intersection -- that cell is (max(qcx0, scx0),
// max(qcy0, scy0)) because the cell map is monotone -- so each pair appears
// exactly once.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "internal.hpp"

namespace april {
namespace {

// Pairs a wave holds in LDS before it appends them (one atomic on the one
// counter each time: per turn of 64 entries, those took longer than the rest).
constexpr uint32_t kHeld = 256;

// A query's rows of cells are dealt out to the waves of `parts` workgroups.
// The entries of a row's cells lie next to each other, so a wave's lanes take
// them side by side, whatever the cells hold; an entry is in its object's
// reporting cell when its place lies between that cell's bounds.  (A thread per
// cell took a large query 0.3 ms and more: its threads walked their cells'
// entries one by one, those of the fullest cell deciding.)
__global__ __launch_bounds__(256) void k_probe(const ProbeQuery *__restrict__ q, uint32_t n_q, uint32_t parts,
                                               const uint32_t *__restrict__ cell_off,
                                               const uint32_t *__restrict__ cell_ids,
                                               const double *__restrict__ boxes,
                                               const uint16_t *__restrict__ cells, uint32_t G,
                                               uint32_t *pr, uint32_t *ps, uint32_t cap,
                                               unsigned int *count) {
    __shared__ uint32_t held[4][kHeld];
    const uint32_t lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    for (uint64_t item = blockIdx.x; item < uint64_t(n_q) * parts; item += gridDim.x) {
        const uint32_t k = uint32_t(item / parts), part = uint32_t(item % parts);
        const ProbeQuery Q = q[k];
        uint32_t n = 0;
        auto append = [&]() {
            unsigned int pos = 0;
            if (lane == 0) pos = atomicAdd(count, n);
            pos = uniform(__shfl(pos, 0));
            wave_lds_sync();
            for (uint32_t i = lane; i < n; i += 64) {
                if (pos + i < cap) {
                    pr[pos + i] = k;
                    ps[pos + i] = held[w][i];
                }
            }
            wave_lds_sync();
            n = 0;
        };
        for (uint32_t cy = Q.cy0 + part * 4 + w; cy <= Q.cy1; cy += 4 * parts) {
            const uint32_t *const row = cell_off + uint64_t(cy) * G;
            const uint32_t e = uniform(row[Q.cx1 + 1]);
            for (uint32_t j0 = uniform(row[Q.cx0]); j0 < e; j0 += 64) {
                const uint32_t j = j0 + lane;
                bool emit = false;
                uint32_t s = 0;
                if (j < e) {
                    s = cell_ids[j];
                    const double *sb = boxes + 4 * uint64_t(s);
                    const uint16_t *sc = cells + 4 * uint64_t(s);
                    const bool meet = Q.x0 <= sb[2] && sb[0] <= Q.x1 && Q.y0 <= sb[3] && sb[1] <= Q.y1;
                    if (meet && max(Q.cy0, uint32_t(sc[1])) == cy) {
                        const uint32_t rx = max(Q.cx0, uint32_t(sc[0]));
                        emit = j >= row[rx] && j < row[rx + 1];
                    }
                }
                const uint64_t mask = __ballot(emit);
                if (emit) held[w][n + uint32_t(__popcll(mask & ((1ull << lane) - 1)))] = s;
                n += uint32_t(__popcll(mask));
                if (n > kHeld - 64) append();
            }
        }
        if (n) append();
    }
}

// blockIdx.y: the query; its workgroups copy its lists, 16 bytes a thread and
// turn where both sides allow it.
__device__ __forceinline__ void copy_list(const uint32_t *__restrict__ from, uint32_t *__restrict__ to, uint64_t n) {
    const uint64_t t = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x, stride = uint64_t(gridDim.x) * blockDim.x;
    uint64_t done = 0;
    if (((reinterpret_cast<uintptr_t>(from) | reinterpret_cast<uintptr_t>(to)) & 15) == 0) {
        const uint64_t n4 = n / 4;
        for (uint64_t i = t; i < n4; i += stride)
            reinterpret_cast<uint4 *>(to)[i] = reinterpret_cast<const uint4 *>(from)[i];
        done = 4 * n4;
    }
    for (uint64_t i = done + t; i < n; i += stride) to[i] = from[i];
}

__global__ __launch_bounds__(256) void k_gather(const QueryLists *__restrict__ lists, uint32_t *as, uint32_t *ae,
                                                uint32_t *fs, uint32_t *fe) {
    const QueryLists q = lists[blockIdx.y];
    copy_list(q.as, as + q.a0, q.na);
    copy_list(q.ae, ae + q.a0, q.na);
    copy_list(q.fs, fs + q.f0, q.nf);
    copy_list(q.fe, fe + q.f0, q.nf);
}

}  // namespace

int launch_gather(const QueryLists *d_lists, uint64_t n, uint32_t *as, uint32_t *ae, uint32_t *fs, uint32_t *fe,
                  hipStream_t stream) {
    for (uint64_t k = 0; k < n; k += 65535) {   // (gridDim.y has 16 bits)
        k_gather<<<dim3(16, uint32_t(std::min<uint64_t>(n - k, 65535))), dim3(256), 0, stream>>>(d_lists + k, as, ae, fs,
                                                                                             fe);
        APRIL_HIP_TRY(hipGetLastError());
    }
    return APRIL_OK;
}

int launch_probe(const ProbeQuery *d_q, uint32_t n_q, const uint32_t *cell_off, const uint32_t *cell_ids,
                 const double *boxes, const uint16_t *cells, uint32_t G, uint32_t *pr, uint32_t *ps,
                 uint32_t cap, unsigned int *count, hipStream_t stream) {
    if (n_q == 0) return APRIL_OK;
    // few queries: several workgroups each
    const uint32_t parts = std::max(1u, std::min(8u, 4096 / n_q));
    k_probe<<<dim3(uint32_t(std::min<uint64_t>(uint64_t(n_q) * parts, 4096))), dim3(256), 0, stream>>>(
        d_q, n_q, parts, cell_off, cell_ids, boxes, cells, G, pr, ps, cap, count);
    APRIL_HIP_TRY(hipGetLastError());
    return APRIL_OK;
}

}  // namespace april
