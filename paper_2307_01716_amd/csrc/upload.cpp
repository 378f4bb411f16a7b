// Host lists to the device: raw, or compressed with their block directories.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <vector>

#include "internal.hpp"

using namespace april;

// Lists that were not validated are checked on the device.  Screening takes
// lists for what april.h asks for; on others (F-intervals outside A, unsorted
// or overlapping intervals) the joins may answer otherwise than the summaries
// would, so those have none.
static int check_sound(april_lists_t *L, const uint32_t *as, const uint32_t *ae, const uint32_t *fs,
                       const uint32_t *fe, hipStream_t s) {
    if (L->sound || L->n == 0) return APRIL_OK;
    unsigned int *d_bad = nullptr, bad[2] = {0, 0};
    if (hipMalloc(reinterpret_cast<void **>(&d_bad), sizeof(bad)) != hipSuccess) {
        (void)hipGetLastError();
        return APRIL_OK;   // not known: no summaries
    }
    hipError_t e = hipMemcpyAsync(d_bad, bad, sizeof(bad), hipMemcpyHostToDevice, s);
    int rc = APRIL_OK;
    if (e == hipSuccess) rc = launch_check_lists(L->n, L->d.off_a, as, ae, L->d.off_f, fs, fe, d_bad, s);
    if (e == hipSuccess && !rc) e = hipMemcpyAsync(bad, d_bad, sizeof(bad), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && !rc) e = hipStreamSynchronize(s);
    (void)hipFree(d_bad);
    if (rc) return rc;
    if (e != hipSuccess) return fail(APRIL_E_HIP, std::string("upload: ") + hipGetErrorString(e));
    L->sound = bad[0] == 0;
    return APRIL_OK;
}

// The summaries of an uploaded collection.  Compressed lists are decoded on
// the device for it, into memory that is given back; without room for that
// they have none.
static int upload_summaries(const april_lists_t *h, april_lists_t *L, hipStream_t s) {
    const bool raw = L->codec == APRIL_CODEC_RAW;
    uint64_t longer = 0;
    for (uint64_t k = 0; k < h->n; k++) longer += h->off_a[k + 1] - h->off_a[k] >= (raw ? kExact : kVbyteSummaryMin);
    if (raw) {
        if (int rc = check_sound(L, L->d.start_a, L->d.end_a, L->d.start_f, L->d.end_f, s)) return rc;
        // (waited for: the copies from pageable memory have landed by now, and
        // a call on another stream would read summaries that are not written yet)
        if (L->sound)
            if (int rc = launch_summaries(L, longer, L->d.start_a, L->d.end_a, L->d.start_f, L->d.end_f, s)) return rc;
        APRIL_HIP_TRY(hipStreamSynchronize(s));
        return APRIL_OK;
    }
    if (!longer) return APRIL_OK;
    const uint64_t na = std::max<uint64_t>(L->n_a, 1), nf = std::max<uint64_t>(L->n_f, 1);
    void *tmp = nullptr;
    if (hipMalloc(&tmp, 8 * (na + nf)) != hipSuccess) {
        (void)hipGetLastError();
        return APRIL_OK;
    }
    uint32_t *as = static_cast<uint32_t *>(tmp), *ae = as + na, *fs = ae + na, *fe = fs + nf;
    int rc = launch_decode_lists(L, false, as, ae, s);
    if (!rc) rc = launch_decode_lists(L, true, fs, fe, s);
    if (!rc) rc = check_sound(L, as, ae, fs, fe, s);
    if (!rc && L->sound) rc = launch_summaries(L, longer, as, ae, fs, fe, s);
    const hipError_t e = hipStreamSynchronize(s);
    (void)hipFree(tmp);
    if (!rc && e != hipSuccess) return fail(APRIL_E_HIP, std::string("summaries: ") + hipGetErrorString(e));
    return rc;
}

extern "C" int april_lists_to_device(const april_lists_t *h, uint32_t codec, void *stream,
                          april_lists_t **out) {
    clear_error();
    if (!h || !out) return fail(APRIL_E_INVALID, "NULL argument");
    if (h->device >= 0) return fail(APRIL_E_INVALID, "lists are already on a device");
    if (codec != APRIL_CODEC_RAW && codec != APRIL_CODEC_VBYTE) return fail(APRIL_E_INVALID, "unknown codec");
    int dev = 0;
    APRIL_HIP_TRY(hipGetDevice(&dev));
    auto *L = new (std::nothrow) april_lists;
    if (!L) return fail(APRIL_E_NOMEM, "out of host memory");
    L->grid = h->grid;
    L->partition_key = h->partition_key;
    L->n = h->n; L->n_a = h->n_a; L->n_f = h->n_f;
    L->device = dev;
    L->codec = codec;
    L->sound = h->sound;
    uint64_t longest = 0;
    for (uint64_t k = 0; k < h->n; k++)
        longest = std::max({longest, h->off_a[k + 1] - h->off_a[k], h->off_f[k + 1] - h->off_f[k]});
    L->max_len = uint32_t(std::min<uint64_t>(longest, 0xfffffffeull));
    auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
    const uint64_t n = h->n;
    const size_t b_off = up(8 * (n + 1));
    // host staging for the compressed form (kept alive in L until freed)
    std::vector<uint64_t> boff_a, boff_f, blk_a, blk_f;
    std::vector<uint8_t> bytes_a, bytes_f;
    std::vector<uint32_t> bval_a, bpos_a, bval_f, bpos_f;
    size_t total = 2 * b_off;
    size_t b_a = 0, b_f = 0, b_ba = 0, b_bf = 0, b_va = 0, b_vf = 0;
    if (codec == APRIL_CODEC_RAW) {
        b_a = up(4 * std::max<uint64_t>(h->n_a, 1));
        b_f = up(4 * std::max<uint64_t>(h->n_f, 1));
        total += 2 * b_a + 2 * b_f;
    } else {
        try {
            for (int t = 0; t < 2; t++) {
                const auto &off = t ? h->off_f : h->off_a;
                const auto &st = t ? h->start_f : h->start_a;
                const auto &en = t ? h->end_f : h->end_a;
                auto &bo = t ? boff_f : boff_a;
                auto &bk = t ? blk_f : blk_a;
                auto &by = t ? bytes_f : bytes_a;
                auto &bv = t ? bval_f : bval_a;
                auto &bp = t ? bpos_f : bpos_a;
                bo.resize(n + 1);
                bk.resize(n + 1);
                by.reserve(size_t((off[n]) * 3));
                for (uint64_t k = 0; k < n; k++) {
                    bo[k] = by.size();
                    bk[k] = bv.size();
                    vbyte_encode(st.data() + off[k], en.data() + off[k], off[k + 1] - off[k], by, bv, bp);
                }
                bo[n] = by.size();
                bk[n] = bv.size();
                if (bv.size() != bp.size()) return fail(APRIL_E_INVALID, "block index mismatch");
                // the decoder reads whole aligned 256-byte windows (+4 bytes)
                for (uint32_t pad = 0; pad < 512; pad++) by.push_back(0);
            }
        } catch (...) {
            delete L;
            return fail(APRIL_E_NOMEM, "out of host memory");
        }
        b_ba = up(bytes_a.size());
        b_bf = up(bytes_f.size());
        b_va = up(4 * std::max<size_t>(bval_a.size(), 1));
        b_vf = up(4 * std::max<size_t>(bval_f.size(), 1));
        total += 4 * b_off + b_ba + b_bf + 2 * b_va + 2 * b_vf;
    }
    hipError_t e = hipMalloc(&L->d.block, total);
    if (e != hipSuccess) {
        delete L;
        return fail(APRIL_E_NOMEM, std::string("hipMalloc lists: ") + hipGetErrorString(e));
    }
    char *p = static_cast<char *>(L->d.block);
    L->d.off_a = reinterpret_cast<uint64_t *>(p); p += b_off;
    L->d.off_f = reinterpret_cast<uint64_t *>(p); p += b_off;
    if (codec == APRIL_CODEC_RAW) {
        L->d.start_a = reinterpret_cast<uint32_t *>(p); p += b_a;
        L->d.end_a = reinterpret_cast<uint32_t *>(p); p += b_a;
        L->d.start_f = reinterpret_cast<uint32_t *>(p); p += b_f;
        L->d.end_f = reinterpret_cast<uint32_t *>(p);
    } else {
        L->d.boff_a = reinterpret_cast<uint64_t *>(p); p += b_off;
        L->d.boff_f = reinterpret_cast<uint64_t *>(p); p += b_off;
        L->d.blk_a = reinterpret_cast<uint64_t *>(p); p += b_off;
        L->d.blk_f = reinterpret_cast<uint64_t *>(p); p += b_off;
        L->d.bytes_a = reinterpret_cast<uint8_t *>(p); p += b_ba;
        L->d.bytes_f = reinterpret_cast<uint8_t *>(p); p += b_bf;
        L->d.bval_a = reinterpret_cast<uint32_t *>(p); p += b_va;
        L->d.bpos_a = reinterpret_cast<uint32_t *>(p); p += b_va;
        L->d.bval_f = reinterpret_cast<uint32_t *>(p); p += b_vf;
        L->d.bpos_f = reinterpret_cast<uint32_t *>(p);
        L->d.n_bytes_a = boff_a[n];
        L->d.n_bytes_f = boff_f[n];
        L->d.n_blk_a = bval_a.size();
        L->d.n_blk_f = bval_f.size();
    }
    L->d.bytes = total;
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto cp = [&](void *dst, const void *src, size_t bytes) -> hipError_t {
        return bytes ? hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s) : hipSuccess;
    };
    hipError_t rc = cp(L->d.off_a, h->off_a.data(), 8 * (n + 1));
    if (rc == hipSuccess) rc = cp(L->d.off_f, h->off_f.data(), 8 * (n + 1));
    if (codec == APRIL_CODEC_RAW) {
        if (rc == hipSuccess) rc = cp(L->d.start_a, h->start_a.data(), 4 * h->n_a);
        if (rc == hipSuccess) rc = cp(L->d.end_a, h->end_a.data(), 4 * h->n_a);
        if (rc == hipSuccess) rc = cp(L->d.start_f, h->start_f.data(), 4 * h->n_f);
        if (rc == hipSuccess) rc = cp(L->d.end_f, h->end_f.data(), 4 * h->n_f);
    } else {
        // the staging vectors die with this call: copy synchronously
        if (rc == hipSuccess) rc = cp(L->d.boff_a, boff_a.data(), 8 * (n + 1));
        if (rc == hipSuccess) rc = cp(L->d.boff_f, boff_f.data(), 8 * (n + 1));
        if (rc == hipSuccess) rc = cp(L->d.blk_a, blk_a.data(), 8 * (n + 1));
        if (rc == hipSuccess) rc = cp(L->d.blk_f, blk_f.data(), 8 * (n + 1));
        if (rc == hipSuccess) rc = cp(L->d.bytes_a, bytes_a.data(), bytes_a.size());
        if (rc == hipSuccess) rc = cp(L->d.bytes_f, bytes_f.data(), bytes_f.size());
        if (rc == hipSuccess) rc = cp(L->d.bval_a, bval_a.data(), 4 * bval_a.size());
        if (rc == hipSuccess) rc = cp(L->d.bpos_a, bpos_a.data(), 4 * bpos_a.size());
        if (rc == hipSuccess) rc = cp(L->d.bval_f, bval_f.data(), 4 * bval_f.size());
        if (rc == hipSuccess) rc = cp(L->d.bpos_f, bpos_f.data(), 4 * bpos_f.size());
        if (rc == hipSuccess) rc = hipStreamSynchronize(s);
    }
    if (rc != hipSuccess) {
        (void)hipFree(L->d.block);
        delete L;
        return fail(APRIL_E_HIP, std::string("upload: ") + hipGetErrorString(rc));
    }
    if (int rs = upload_summaries(h, L, s)) {
        april_lists_free(L);
        return rs;
    }
    *out = L;
    return APRIL_OK;
}
