// C ABI of libdtans (declared in include/dtans.h).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <chrono>
#include <string>
#include <vector>

#include "container.hpp"
#include "dtans.h"
#include "kernels.hpp"
#include "launch_plan.hpp"

using namespace dtans;

namespace dtans {
// sym_kernels.hip: sums[i] = beta * y[i] + alpha * d[i] * x[i] (d null: beta *
// y[i]), in y itself with FP64 or without sums; y[i] = sums[i]
hipError_t launch_sym_start(bool f64, const void *d, const void *x, void *y, double *sums, int64_t n, double alpha,
                            double beta, hipStream_t st);
hipError_t launch_sym_end(const double *sums, float *y, int64_t n, hipStream_t st);
}  // namespace dtans

namespace {

thread_local std::string g_last_error;

dtans_status set_err(dtans_status s, const std::string &msg) {
    g_last_error = msg;
    return s;
}

dtans_status from_msg(const std::string &m) {
    if (m.empty()) return DTANS_OK;
    struct { const char *p; dtans_status s; } map[] = {
        {"EINVAL", DTANS_EINVAL}, {"EUNSORTED", DTANS_EUNSORTED}, {"ERANGE", DTANS_ERANGE},
        {"ENOMEM", DTANS_ENOMEM}, {"ECORRUPT", DTANS_ECORRUPT}, {"EIO", DTANS_EIO},
        {"EUNSUPPORTED", DTANS_EUNSUPPORTED}, {"EHIP", DTANS_EHIP}};
    for (auto &e : map)
        if (m.compare(0, strlen(e.p), e.p) == 0 && m.size() > strlen(e.p) && m[strlen(e.p)] == ':')
            return set_err(e.s, m);
    return set_err(DTANS_EINVAL, m);
}

dtans_status hip_err(hipError_t e, const char *what) {
    return set_err(DTANS_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(call)                                            \
    do {                                                         \
        hipError_t e_ = (call);                                  \
        if (e_ != hipSuccess) return hip_err(e_, #call);         \
    } while (0)

int device_cus(int dev) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    return cus;
}

// Device memory owned by a handle; freed in one place.
struct DevBufs {
    std::vector<void *> ptrs;
    uint8_t *pool = nullptr;  // of reserve: what is left of one allocation for several buffers
    size_t pool_left = 0;
    ~DevBufs() { release(); }
    void release() {
        for (void *p : ptrs) (void)hipFree(p);
        ptrs.clear();
        pool = nullptr;
        pool_left = 0;
    }
    static size_t padded(size_t bytes, size_t pad = 256) { return (bytes + pad + 255) / 256 * 256; }
    // a piece of what reserve allocated, as it is
    void *take(size_t bytes) {
        const size_t size = padded(bytes, 0);
        if (size == 0 || size > pool_left) return nullptr;
        void *p = pool;
        pool += size;
        pool_left -= size;
        return p;
    }
    // one allocation for the uploads that follow (the sum of their padded sizes)
    hipError_t reserve(size_t bytes) {
        void *p = nullptr;
        hipError_t e = hipMalloc(&p, bytes);
        if (e != hipSuccess) return e;
        ptrs.push_back(p);
        pool = (uint8_t *)p;
        pool_left = bytes;
        return hipSuccess;
    }
    // copy `bytes` from host (or zero-fill when src is null) into a new buffer
    // padded by `pad` zero bytes
    hipError_t upload(void **dst, const void *src, size_t bytes, hipStream_t st, size_t pad = 256) {
        void *p = nullptr;
        hipError_t e = hipSuccess;
        const size_t size = padded(bytes, pad);
        if (size <= pool_left) {
            p = pool;
            pool += size;
            pool_left -= size;
        } else {
            e = hipMalloc(&p, size);
            if (e != hipSuccess) return e;
            ptrs.push_back(p);
        }
        const size_t from = src ? bytes : 0;
        e = hipMemsetAsync((uint8_t *)p + from, 0, size - from, st);
        if (e != hipSuccess) return e;
        if (src && bytes) e = hipMemcpyAsync(p, src, bytes, hipMemcpyHostToDevice, st);
        *dst = p;
        return e;
    }
};

}  // namespace

namespace dtans {
// the thread-local error message, for the library's other source files
dtans_status set_error(dtans_status s, const std::string &msg) { return set_err(s, msg); }
}  // namespace dtans

namespace {
}  // namespace

struct dtans_matrix {
    Container c;
    std::vector<uint64_t> gtab;
    std::vector<uint8_t> gval;
    std::vector<int32_t> lane_row, split_row, split_first, split_last, split_long;
    std::vector<int32_t> nzr, empty_rows;  // layout NNZ: {row, end} pairs; rows without nonzeros
    DevBufs bufs;
    bool uploaded = false;
    int device = -1, num_cus = 256;
    int waves_per_wg = 0, wg_per_cu = 0, stage = 0;
    bool one_walk = false;  // see Launch
    DevMat view{};
    std::vector<uint32_t> escv32;  // FP32 escaped values as uploaded (kept with the handle)
    std::vector<int32_t> orig_row_ptr;  // row-sorted containers: the original matrix's row pointers
    // device scratch of the products (layout NNZ partial sums, the transposed
    // product's per-CU copies of dX, the FP32 symmetric product's sums); sized
    // by dtans_to_device (a piece of the matrix's own allocation) / dtans_reserve
    void *scratch = nullptr;
    size_t scratch_bytes = 0;
    bool scratch_in_bufs = false;
    int32_t reserved_k = 0;
};

struct dtans_batch {
    std::vector<dtans_matrix *> mats;
    bool f64 = true;
    DevBufs bufs;
    BatchDev dev{};
    Launch launch{};
    std::vector<BatchTask> tasks;
    std::vector<int32_t> wg_task;
};

struct dtans_csr {
    int64_t m = 0, n = 0, nnz = 0;
    bool f64 = true;
    DevBufs bufs;
    CsrDev dev{};
    int device = -1, num_cus = 256;
    double *partial = nullptr;  // variant 2: partial sums (owned by bufs)
    int64_t bytes = 0;
};

namespace {

// split rows spanning more lanes than one thread should sum (the fix-up's
// kLongSplit, 4 following lanes)
std::vector<int32_t> long_splits(const std::vector<int32_t> &first, const std::vector<int32_t> &last,
                                 int limit) {
    std::vector<int32_t> out;
    for (size_t s = 0; s < first.size(); ++s)
        if (last[s] - first[s] > limit) out.push_back((int32_t)s);
    return out;
}

// Layout NNZ: the list of nonempty rows as {row, end} pairs with a {m, nnz}
// sentinel, the rows without nonzeros, and lane_row rewritten from a row to
// its index in the list (a lane's first nonzero always lies in a nonempty row).
void nonempty_rows(const Container &c, std::vector<int32_t> &lane_row, std::vector<int32_t> &nzr,
                   std::vector<int32_t> &empty) {
    nzr.clear();
    empty.clear();
    if (c.layout != kLayoutNnz) return;
    std::vector<int32_t> index(c.m, -1);
    for (int64_t i = 0; i < c.m; ++i) {
        if (c.row_ptr[i] < c.row_ptr[i + 1]) {
            index[i] = (int32_t)(nzr.size() / 2);
            nzr.push_back((int32_t)i);
            nzr.push_back(c.row_ptr[i + 1]);
        } else {
            empty.push_back((int32_t)i);
        }
    }
    nzr.push_back((int32_t)c.m);
    nzr.push_back((int32_t)c.nnz);
    for (auto &r : lane_row) {
        // lane 0 is listed at row 0, which may be empty: its first nonzero
        // lies in the first nonempty row
        int64_t i = r;
        while (i < c.m && index[i] < 0) ++i;
        r = i < c.m ? index[i] : (int32_t)(nzr.size() / 2 - 1);
    }
}

// SpMV stages its streams through an LDS ring only when asked to (measured:
// the direct-read kernels, at twice the waves per SIMD, are faster on the
// workloads here); a wavefront's run of streams is addressed with 32-bit
// offsets.  Streams with escapes inside them are read directly: a step may
// read more of such a stream than the ring keeps ahead of it.
bool uses_ring(const dtans_matrix *h) {
    return h->stage == DTANS_STAGE_RING && h->c.esc_mode == 0 && 4 * (int64_t)h->c.words.size() < (1ll << 31);
}

// Whether the decode to CSR takes one walk rather than two (row layout).  Two
// walks write whole cache lines together, which pays while all lanes of a wave
// decode; one keeps 32 waves a CU resident instead of 16 and has the shorter
// chain, which pays where the longest rows of the waves, each a serial chain,
// take longer than writing the matrix (0.13 us a nonzero against 2.4 TB/s).
// A million skewed rows of mean 12 to 17, FP32, longest row 100 (chains 0.8 of
// the bound below): 105 us in two walks, 119 in one; 200 (1.2): 172, 156; 1000:
// 546, 372; rows of 12: 52, 97.  A long row among regular ones, which leaves
// most lanes busy, is no reason (one of 2669 in 2,000,000 of 12: 411, 465).
// With no more waves than two walks keep resident only much longer rows count
// (200,000 rows, longest 200: 51, 53; 2000: 289, 269; below 64 times the mean
// 0.94 to 1.05).  Sorted rows are written apart from each other, and their
// long waves come a window apart, all to the same wavefronts: one walk with
// more waves than are resident (1,000,000 rows, longest 500, windows of 256,
// FP32: 374, 250), FP64 from the smallest matrix on (2000 rows: 34, 32).
bool takes_one_walk(const Container &c, int num_cus) {
    if (c.layout != kLayoutRow || c.m == 0) return false;
    const int64_t resident = 16ll * num_cus;
    if (c.sigma && (c.dtype == kF64 || c.num_waves > resident)) return true;
    int64_t longest = 0, chains = 0;
    for (int64_t w = 0; w < c.m; w += 64) {
        const int32_t *r = c.row_ptr.data() + w;
        const int rows = (int)std::min<int64_t>(c.m - w, 64);
        int32_t most = 0;
        for (int i = 0; i < rows; ++i) most = std::max(most, r[i + 1] - r[i]);
        longest = std::max<int64_t>(longest, most);
        chains += most;
    }
    if (64 * chains < 2 * c.nnz) return false;
    if (c.num_waves <= resident && longest <= 64 * std::max<int64_t>(c.nnz / c.m, 4)) return false;
    return std::max(longest, chains / resident) * 27000 > c.nnz;
}

Launch plan_launch(const dtans_matrix *h) {
    const ShapePlan sp = plan_shape(h->c.dtype == kF64, h->c.layout == kLayoutRow, h->waves_per_wg, h->wg_per_cu);
    const int wpw = sp.waves_per_wg, wgcu = sp.wg_per_cu;
    Launch L;
    L.waves_per_wg = wpw;
    int64_t need = (h->c.num_waves + wpw - 1) / wpw;
    int64_t grid = (int64_t)h->num_cus * wgcu;
    L.grid = (int)std::max<int64_t>(1, std::min(grid, need));
    L.num_cus = h->num_cus;
    L.ring = uses_ring(h) ? 1 : 0;
    // ring kernels: 16-wave workgroups unless set, as many per CU as fit
    L.ring_waves_per_wg = h->waves_per_wg > 0 ? h->waves_per_wg : 16;
    L.wg_per_cu = h->wg_per_cu;
    L.fixed_shape = sp.fixed ? 1 : 0;
    L.one_walk = h->one_walk ? 1 : 0;
    return L;
}

// FP64 sums of the FP32 symmetric product (FP64 adds into y itself)
size_t sym_sums_bytes(const Container &c) {
    return c.dtype == kF64 || c.m != c.n || c.sigma || c.nnz == 0 ? 0 : sizeof(double) * (size_t)c.n;
}

// scratch a product with up to k right-hand sides needs (either direction)
size_t scratch_need(const dtans_matrix *h, int32_t k) {
    const bool f64 = h->c.dtype == kF64;
    const size_t a = spmm_scratch_bytes(h->view, k);
    const size_t b = h->c.nnz > 0 ? spmm_t_work_bytes(h->view, f64, h->num_cus) : 0;
    return std::max(std::max(a, b), sym_sums_bytes(h->c));
}

dtans_status upload(dtans_matrix *h, hipStream_t st) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (h->uploaded) {
        if (dev != h->device)
            return set_err(DTANS_EINVAL, "matrix was uploaded to device " + std::to_string(h->device) +
                                             ", current device is " + std::to_string(dev));
        return DTANS_OK;
    }
    const Container &c = h->c;
    const bool direct = gpu_table(c, h->gtab, h->gval);
    nnz_layout_meta(c, h->lane_row, h->split_row, h->split_first, h->split_last);
    nonempty_rows(c, h->lane_row, h->nzr, h->empty_rows);
    h->split_long = long_splits(h->split_first, h->split_last, kLongSplitRuns);
    const bool f64 = c.dtype == kF64;
    const void *escv_src = c.escv.data();
    size_t escv_bytes = c.escv.size() * 8;
    if (!f64) {
        h->escv32.resize(c.escv.size());
        for (size_t i = 0; i < c.escv.size(); ++i) h->escv32[i] = (uint32_t)c.escv[i];
        escv_src = h->escv32.data();
        escv_bytes = h->escv32.size() * 4;
    }
    void *p[18];
    if (c.sigma && !original_row_ptr(c, h->orig_row_ptr)) return set_err(DTANS_ECORRUPT, "bad row order");
    struct Part {
        const void *src;
        size_t bytes;
    };
    std::vector<Part> parts = {
        {h->gtab.data(), 8 * h->gtab.size()},           {h->gval.data(), h->gval.size()},
        {c.row_ptr.data(), 4 * c.row_ptr.size()},       {c.word_off.data(), 8 * c.word_off.size()},
        {c.escd_off.data(), 8 * c.escd_off.size()},     {c.escv_off.data(), 8 * c.escv_off.size()},
        {c.words.data(), 4 * c.words.size()},           {c.escd.data(), 4 * c.escd.size()},
        {escv_src, escv_bytes},                         {h->lane_row.data(), 4 * h->lane_row.size()},
        {h->split_row.data(), 4 * h->split_row.size()}, {h->split_first.data(), 4 * h->split_first.size()},
        {h->split_last.data(), 4 * h->split_last.size()}, {h->nzr.data(), 4 * h->nzr.size()},
        {h->empty_rows.data(), 4 * h->empty_rows.size()}, {h->split_long.data(), 4 * h->split_long.size()}};
    if (c.sigma) {
        parts.push_back({c.perm.data(), 4 * c.perm.size()});
        parts.push_back({h->orig_row_ptr.data(), 4 * h->orig_row_ptr.size()});
    }
    DevMat &v = h->view;
    v.m = c.m;
    v.n = c.n;
    v.nnz = c.nnz;
    v.num_lanes = c.num_lanes;
    v.num_waves = c.num_waves;
    v.lane_nnz = (int32_t)c.lane_nnz;
    v.layout = (int32_t)c.layout;
    h->num_cus = device_cus(dev);
    // the scratch of one right-hand side lies behind the matrix: an allocation
    // of its own costs 0.2 ms
    const size_t scratch = scratch_need(h, 1);
    size_t total = DevBufs::padded(scratch, 0);
    for (const Part &q : parts) total += DevBufs::padded(q.bytes);
    HIP_TRY(h->bufs.reserve(total));
    p[16] = p[17] = nullptr;
    for (size_t i = 0; i < parts.size(); ++i) HIP_TRY(h->bufs.upload(&p[i], parts[i].src, parts[i].bytes, st));
    // the copies complete before the call returns, so that products on any
    // stream find the matrix in place (the one synchronisation of a handle)
    HIP_TRY(hipStreamSynchronize(st));
    if (!h->scratch && scratch > 0) {
        h->scratch = h->bufs.take(scratch);
        h->scratch_bytes = h->scratch ? scratch : 0;
        h->scratch_in_bufs = h->scratch != nullptr;
    }
    v.tab = (const uint64_t *)p[0];
    v.tabval = p[1];
    v.row_ptr = (const int32_t *)p[2];
    v.woff = (const uint64_t *)p[3];
    v.doff = (const uint64_t *)p[4];
    v.voff = (const uint64_t *)p[5];
    v.words = (const uint32_t *)p[6];
    v.escd = (const uint32_t *)p[7];
    v.escv = p[8];
    v.lane_row = (const int32_t *)p[9];
    v.nzr = (const int2 *)p[13];
    v.empty_rows = (const int32_t *)p[14];
    v.n_nzr = c.layout == kLayoutNnz ? (int64_t)h->nzr.size() / 2 - 1 : 0;
    v.n_empty = (int64_t)h->empty_rows.size();
    v.split.row = (const int32_t *)p[10];
    v.split.first = (const int32_t *)p[11];
    v.split.last = (const int32_t *)p[12];
    v.split.longs = (const int32_t *)p[15];
    v.split.n = (int64_t)h->split_row.size();
    v.split.n_long = (int64_t)h->split_long.size();
    v.base_direct = direct ? 1 : 0;
    v.no_escape = c.dtab.has_escape || c.vtab.has_escape ? 0 : 1;
    v.first_mode = c.first_mode;
    v.esc_in_stream = c.esc_mode == 1 ? 1 : 0;
    v.row_perm = c.sigma ? (const int32_t *)p[16] : nullptr;
    v.orig_row_ptr = c.sigma ? (const int32_t *)p[17] : nullptr;
    h->device = dev;
    h->one_walk = takes_one_walk(c, h->num_cus);
    h->uploaded = true;
    return DTANS_OK;
}

// Upload if needed, then grow the scratch to what products with up to k
// right-hand sides need.  Growing waits for the device (earlier launches on
// any stream may still read the old buffer) before the old one is freed.
dtans_status reserve(dtans_matrix *h, int32_t k, hipStream_t st) {
    dtans_status s = upload(h, st);
    if (s) return s;
    if (k <= h->reserved_k) return DTANS_OK;
    const size_t need = scratch_need(h, k);
    if (need > h->scratch_bytes) {
        if (h->scratch) {
            HIP_TRY(hipDeviceSynchronize());
            if (!h->scratch_in_bufs) HIP_TRY(hipFree(h->scratch));
            h->scratch = nullptr;
            h->scratch_bytes = 0;
            h->scratch_in_bufs = false;
        }
        HIP_TRY(hipMalloc(&h->scratch, need));
        h->scratch_bytes = need;
    }
    h->reserved_k = std::max(h->reserved_k, std::min(k, kMaxPassCols));
    if (k > kMaxPassCols) h->reserved_k = k;  // wider products reuse the pass-wide scratch
    return DTANS_OK;
}

// Product calls allocate and synchronise nothing: the matrix must be on the
// current device (dtans_to_device) with scratch for k columns (dtans_reserve;
// dtans_to_device reserves for k = 1).
dtans_status ready(dtans_matrix *h, int32_t k) {
    if (!h) return set_err(DTANS_EINVAL, "null matrix handle");
    if (!h->uploaded) return set_err(DTANS_EINVAL, "matrix is not on the device: call dtans_to_device first");
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != h->device)
        return set_err(DTANS_EINVAL, "matrix was uploaded to device " + std::to_string(h->device) +
                                         ", current device is " + std::to_string(dev));
    if (k > 0 && scratch_need(h, k) > h->scratch_bytes)
        return set_err(DTANS_EINVAL, "scratch reserved for fewer right-hand sides: call dtans_reserve(" +
                                         std::to_string(k) + ") first");
    return DTANS_OK;
}

int64_t sell_bytes(const Container &c, int slice) {
    int64_t total = 4 * ((c.m + slice - 1) / slice + 1);
    const int64_t per = 4 + (int64_t)c.value_bytes();
    for (int64_t s = 0; s < c.m; s += slice) {
        int64_t mx = 0;
        for (int64_t i = s; i < std::min(c.m, s + slice); ++i)
            mx = std::max<int64_t>(mx, c.row_ptr[i + 1] - c.row_ptr[i]);
        total += slice * mx * per;
    }
    return total;
}

// Resolve layout AUTO and lane_nnz 0 the way dtans_encode_csr does.  One row
// per lane unless the rows are long or irregular enough that 64-row waves
// would be too few or badly balanced; for the nonzero layout an encoded wave,
// or four for irregular rows, for every wavefront that 256 CUs keep resident
// (six per SIMD), 32..512 nonzeros a lane.
void auto_encoding(int64_t m, int64_t nnz, const int32_t *row_ptr, const dtans_encode_opts &o,
                   bool f64, int &layout, int &T) {
    layout = o.layout;
    int64_t maxlen = 0;
    for (int64_t i = 0; i < m; ++i) maxlen = std::max<int64_t>(maxlen, row_ptr[i + 1] - row_ptr[i]);
    const double mean = m ? (double)nnz / m : 0;
    if (layout == DTANS_LAYOUT_AUTO) {
        int64_t waves = (m + 63) / 64;
        layout = (waves < 2048 || maxlen > 8 * std::max(mean, 4.0)) ? DTANS_LAYOUT_NNZ : DTANS_LAYOUT_ROW;
    }
    T = 0;
    if (layout == DTANS_LAYOUT_NNZ) {
        T = o.lane_nnz;
        if (T == 0) {
            // wavefronts the SpMV launch keeps resident on 256 CUs
            int wpw = 0, wgcu = 0;
            default_shape(f64, kNnzWavesPerSimd, wpw, wgcu);
            const int64_t resident = 256LL * wpw * wgcu;
            int64_t t;
            if (maxlen <= 4 * std::max(mean, 1.0)) {
                // regular rows: encoded waves cost about the same, so give
                // every resident wavefront exactly one of them: a second,
                // partial round would double the time of a share
                t = (nnz + 64 * resident - 1) / (64 * resident);
            } else {
                // irregular rows: the cost of a wave varies with its rows;
                // about four per wavefront even it out (R-MAT scale 22:
                // 0.574 ms at 4.3 waves per wavefront, 0.617 at 1.3)
                t = nnz / (64 * resident * 4);
            }
            T = (int)std::min<int64_t>(512, std::max<int64_t>(32, (t + 3) / 4 * 4));
        }
    }
}

// Launch shapes for one encoding: workgroups per CU from the LDS limit down to
// 1, waves per workgroup filling the CU's wave slots, then half and a quarter.
std::vector<std::pair<int, int>> launch_shapes(int layout, bool f64, int wpw_fixed, int wg_fixed) {
    const int table_bytes = kSlots * (8 + (f64 ? 8 : 4));
    const int maxwg = std::max(1, 160 * 1024 / table_bytes);
    const int per_simd = layout == DTANS_LAYOUT_ROW ? kRowWavesPerSimd : kNnzWavesPerSimd;
    std::vector<std::pair<int, int>> out;  // (waves_per_wg, wg_per_cu)
    std::vector<int> wgs;
    if (wg_fixed) {
        wgs.push_back(wg_fixed);
    } else {
        // the library's own shape first (launched as without options)
        int dw = 0, dg = 0;
        default_shape(f64, per_simd, dw, dg);
        if (!wpw_fixed) out.push_back({dw, dg});
        wgs.push_back(dg);
        for (int g = maxwg; g >= 1; --g)
            if (g != dg) wgs.push_back(g);
    }
    for (int g : wgs) {
        // waves dealt evenly to the 4 SIMDs (see default_shape)
        const int base = std::min(16, std::max(4, (4 * per_simd / g) & ~3));
        std::vector<int> ws;
        if (wpw_fixed) ws.push_back(wpw_fixed);
        else
            for (int w : {base, base / 2, base / 4})
                if (w >= 2 && std::find(ws.begin(), ws.end(), w) == ws.end()) ws.push_back(w);
        for (int w : ws)
            if (std::find(out.begin(), out.end(), std::make_pair(w, g)) == out.end()) out.push_back({w, g});
    }
    return out;
}

dtans_status tune_candidates(int64_t m, int64_t nnz, const int32_t *row_ptr, dtans_dtype dtype,
                             int32_t k, const dtans_encode_opts *in,
                             std::vector<dtans_encode_opts> &out) {
    out.clear();
    if (!in || !row_ptr) return set_err(DTANS_EINVAL, "null argument");
    if (m < 0 || nnz < 0) return set_err(DTANS_EINVAL, "negative size");
    if (m >= (1ll << 31) || nnz >= (1ll << 31))
        return set_err(DTANS_ERANGE, "rows and nonzeros must be below 2^31");
    if (dtype != DTANS_F32 && dtype != DTANS_F64) return set_err(DTANS_EINVAL, "dtype must be F32 or F64");
    if (k < 1) return set_err(DTANS_EINVAL, "k must be >= 1");
    const dtans_encode_opts &o = *in;
    if (o.layout < DTANS_LAYOUT_AUTO || o.layout > DTANS_LAYOUT_NNZ)
        return set_err(DTANS_EINVAL, "layout must be AUTO, ROW or NNZ");
    if (o.lane_nnz < 0 || o.lane_nnz % 4) return set_err(DTANS_EINVAL, "lane_nnz must be a multiple of 4");
    if (o.waves_per_wg < 0 || o.waves_per_wg > 16 || o.wg_per_cu < 0 || o.wg_per_cu > 32)
        return set_err(DTANS_EINVAL, "waves_per_wg must be 0..16 and wg_per_cu 0..32");
    if (row_ptr[0] != 0 || row_ptr[m] != nnz) return set_err(DTANS_EINVAL, "row_ptr must run from 0 to nnz");
    for (int64_t i = 0; i < m; ++i)
        if (row_ptr[i + 1] < row_ptr[i]) return set_err(DTANS_EINVAL, "row_ptr decreases");
    // encodings: the automatic choice first, then the other layout, then
    // neighbouring lane lengths (x1/2, x2, x1/4, x4 of the automatic one)
    int auto_layout = 0, auto_T = 0;
    auto_encoding(m, nnz, row_ptr, o, dtype == DTANS_F64, auto_layout, auto_T);
    std::vector<std::pair<int, int>> enc{{auto_layout, auto_T}};
    auto add = [&](int lay, int T) {
        for (auto &e : enc)
            if (e.first == lay && e.second == T) return;
        enc.push_back({lay, T});
    };
    if (o.layout == DTANS_LAYOUT_AUTO) {
        dtans_encode_opts nn = o;
        nn.layout = DTANS_LAYOUT_NNZ;
        int lay = 0, T0 = 0;
        auto_encoding(m, nnz, row_ptr, nn, dtype == DTANS_F64, lay, T0);
        add(DTANS_LAYOUT_ROW, 0);
        add(DTANS_LAYOUT_NNZ, T0);
    }
    const bool nnz_possible = o.layout != DTANS_LAYOUT_ROW;
    if (nnz_possible && o.lane_nnz == 0) {
        dtans_encode_opts nn = o;
        nn.layout = DTANS_LAYOUT_NNZ;
        int lay = 0, T0 = 0;
        auto_encoding(m, nnz, row_ptr, nn, dtype == DTANS_F64, lay, T0);
        for (int f : {-2, 2, -4, 4}) {
            int T = f > 0 ? T0 * f : T0 / -f;
            T = std::min(512, std::max(32, (T + 3) / 4 * 4));
            add(DTANS_LAYOUT_NNZ, T);
        }
    }
    if (o.stream_stage < 0 || o.stream_stage > DTANS_STAGE_RING)
        return set_err(DTANS_EINVAL, "stream_stage must be 0, 1 or 2");
    for (auto &e : enc) {
        auto push = [&](int w, int g, int stage) {
            dtans_encode_opts c = o;
            c.layout = e.first;
            c.lane_nnz = e.second;
            if (c.layout == DTANS_LAYOUT_NNZ) c.sort_window = 0;  // row sorting is a ROW-layout option
            c.waves_per_wg = w;
            c.wg_per_cu = g;
            c.stream_stage = stage;
            out.push_back(c);
        };
        // the direct-read shapes, then the LDS-ring kernels (their own
        // shapes; workgroups per CU as many as fit unless fixed)
        if (o.stream_stage != DTANS_STAGE_RING)
            for (auto &w : launch_shapes(e.first, dtype == DTANS_F64, o.waves_per_wg, o.wg_per_cu))
                push(w.first, w.second, DTANS_STAGE_DIRECT);
        if (o.stream_stage != DTANS_STAGE_DIRECT) {
            if (o.waves_per_wg) push(o.waves_per_wg, o.wg_per_cu, DTANS_STAGE_RING);
            else
                for (int w : {16, 8, 4}) push(w, o.wg_per_cu, DTANS_STAGE_RING);
        }
    }
    return DTANS_OK;
}

// 64-bit FNV-1a over 8-byte words (a fingerprint, not a checksum of record)
struct Fingerprint {
    uint64_t h = 0xcbf29ce484222325ull;
    void word(uint64_t w) {
        h ^= w;
        h *= 0x100000001b3ull;
    }
    void bytes(const void *p, size_t n) {
        const uint8_t *b = (const uint8_t *)p;
        size_t i = 0;
        for (; i + 8 <= n; i += 8) {
            uint64_t w;
            memcpy(&w, b + i, 8);
            word(w);
        }
        uint64_t t = 0;
        memcpy(&t, b + i, n - i);
        word(t ^ ((uint64_t)(n - i) << 56));
    }
};

struct TuneResources {
    hipStream_t st = nullptr;
    std::vector<hipEvent_t> ev;
    DevBufs bufs;
    dtans_matrix *h = nullptr;
    ~TuneResources() {
        if (st) (void)hipStreamSynchronize(st);
        if (h) dtans_destroy(h);
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
        bufs.release();
        if (st) (void)hipStreamDestroy(st);
    }
};

}  // namespace

extern "C" {

const char *dtans_version(void) { return "dtans 0.1.0 (gfx950, CSR-dtANS container v1)"; }

const char *dtans_last_error(void) { return g_last_error.c_str(); }

void dtans_default_opts(dtans_encode_opts *o) {
    if (!o) return;
    memset(o, 0, sizeof(*o));
    o->layout = DTANS_LAYOUT_AUTO;
    o->perm_seed = 1;
}

namespace {

dtans_status encode_common(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr,
                           const int32_t *col_idx, const void *vals, dtans_dtype dtype,
                           const dtans_encode_opts *opts, DeviceEncoder *dev, dtans_matrix **out) {
    if (!out) return set_err(DTANS_EINVAL, "out is null");
    *out = nullptr;
    dtans_encode_opts o;
    dtans_default_opts(&o);
    if (opts) o = *opts;
    if (m < 0 || n < 0 || nnz < 0) return set_err(DTANS_EINVAL, "negative size");
    if (m >= (1ll << 31) || n >= (1ll << 31) || nnz >= (1ll << 31))
        return set_err(DTANS_ERANGE, "rows, columns and nonzeros must be below 2^31");
    if (!row_ptr || (nnz > 0 && (!col_idx || !vals))) return set_err(DTANS_EINVAL, "null array");
    if (o.waves_per_wg < 0 || o.waves_per_wg > 16 || o.wg_per_cu < 0 || o.wg_per_cu > 32)
        return set_err(DTANS_EINVAL, "waves_per_wg must be 0..16 and wg_per_cu 0..32");
    if (o.stream_stage < 0 || o.stream_stage > DTANS_STAGE_RING)
        return set_err(DTANS_EINVAL, "stream_stage must be 0, 1 or 2");
    if (o.max_mult < 0 || o.max_mult > kMaxBase)
        return set_err(DTANS_EINVAL, "max_mult must be 0..256");
    if (o.escape_in_stream != 0 && o.escape_in_stream != 1)
        return set_err(DTANS_EINVAL, "escape_in_stream must be 0 or 1");
    if (o.sort_window < 0 || o.sort_window % 64)
        return set_err(DTANS_EINVAL, "sort_window must be 0 or a positive multiple of 64");
    const size_t vb = dtype == DTANS_F64 ? 8 : 4;
    std::vector<int32_t> scol;
    std::vector<uint8_t> sval;
    if (o.sort_rows && nnz > 0) {
        if (row_ptr[0] != 0 || row_ptr[m] != nnz) return set_err(DTANS_EINVAL, "row_ptr must run from 0 to nnz");
        scol.assign(col_idx, col_idx + nnz);
        sval.assign((const uint8_t *)vals, (const uint8_t *)vals + nnz * vb);
        std::vector<int64_t> idx;
        for (int64_t i = 0; i < m; ++i) {
            if (row_ptr[i + 1] < row_ptr[i]) return set_err(DTANS_EINVAL, "row_ptr decreases");
            int64_t b = row_ptr[i], e = row_ptr[i + 1];
            idx.resize(e - b);
            for (int64_t q = b; q < e; ++q) idx[q - b] = q;
            std::stable_sort(idx.begin(), idx.end(),
                             [&](int64_t a, int64_t c) { return col_idx[a] < col_idx[c]; });
            for (int64_t q = b; q < e; ++q) {
                scol[q] = col_idx[idx[q - b]];
                memcpy(&sval[q * vb], (const uint8_t *)vals + idx[q - b] * vb, vb);
            }
        }
        col_idx = scol.data();
        vals = sval.data();
    }
    EncodeParams p;
    p.seed = o.perm_seed;
    p.max_mult = o.max_mult ? (uint32_t)o.max_mult : 255u;
    p.first_mode = o.first_delta_column ? 0u : 1u;
    p.esc_mode = o.escape_in_stream ? 1u : 0u;
    p.sigma = (uint32_t)o.sort_window;
    if (o.sort_window && o.layout == DTANS_LAYOUT_AUTO) o.layout = DTANS_LAYOUT_ROW;
    int layout = 0, T = 0;
    auto_encoding(m, nnz, row_ptr, o, dtype == DTANS_F64, layout, T);
    p.layout = layout == DTANS_LAYOUT_NNZ ? kLayoutNnz : kLayoutRow;
    if (p.layout == kLayoutNnz) p.lane_nnz = (uint32_t)T;
    dtans_matrix *h = new dtans_matrix();
    std::string err = encode_csr(m, n, nnz, row_ptr, col_idx, vals, dtype, p, h->c, dev);
    if (!err.empty()) {
        delete h;
        return from_msg(err);
    }
    h->waves_per_wg = o.waves_per_wg;
    h->wg_per_cu = o.wg_per_cu;
    h->stage = o.stream_stage;
    *out = h;
    return DTANS_OK;
}

}  // namespace

dtans_status dtans_encode_csr(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr,
                              const int32_t *col_idx, const void *vals, dtans_dtype dtype,
                              const dtans_encode_opts *opts, dtans_matrix **out) {
    return encode_common(m, n, nnz, row_ptr, col_idx, vals, dtype, opts, nullptr, out);
}

dtans_status dtans_encode_csr_gpu(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr,
                                  const int32_t *col_idx, const void *vals, dtans_dtype dtype,
                                  const dtans_encode_opts *opts, void *stream, dtans_matrix **out) {
    std::unique_ptr<DeviceEncoder> dev(new_device_encoder(stream));
    return encode_common(m, n, nnz, row_ptr, col_idx, vals, dtype, opts, dev.get(), out);
}

dtans_status dtans_encode_csr_device(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr,
                                     const int32_t *col_idx, const void *vals, dtans_dtype dtype,
                                     const dtans_encode_opts *opts, void *stream, dtans_matrix **out) {
    if (!out) return set_err(DTANS_EINVAL, "out is null");
    *out = nullptr;
    if (m < 0 || n < 0 || nnz < 0) return set_err(DTANS_EINVAL, "negative size");
    if (m >= (1ll << 31) || n >= (1ll << 31) || nnz >= (1ll << 31))
        return set_err(DTANS_ERANGE, "rows, columns and nonzeros must be below 2^31");
    if (!row_ptr || (nnz > 0 && (!col_idx || !vals))) return set_err(DTANS_EINVAL, "null array");
    if (opts && opts->sort_rows) return set_err(DTANS_EUNSUPPORTED, "sort_rows needs host arrays");
    hipStream_t st = (hipStream_t)stream;
    std::vector<int32_t> rp(m + 1);
    HIP_TRY(hipMemcpyAsync(rp.data(), row_ptr, (m + 1) * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    std::unique_ptr<DeviceEncoder> dev(new_device_encoder(stream, true));
    return encode_common(m, n, nnz, rp.data(), col_idx, vals, dtype, opts, dev.get(), out);
}

dtans_status dtans_save(const dtans_matrix *mat, const char *path) {
    if (!mat || !path) return set_err(DTANS_EINVAL, "null argument");
    return from_msg(save_container(mat->c, path));
}

dtans_status dtans_load(const char *path, dtans_matrix **out) {
    if (!path || !out) return set_err(DTANS_EINVAL, "null argument");
    *out = nullptr;
    dtans_matrix *h = new dtans_matrix();
    std::string err = load_container(path, h->c);
    if (err.empty()) err = host_decode(h->c, nullptr, nullptr);
    if (!err.empty()) {
        delete h;
        return from_msg(err);
    }
    *out = h;
    return DTANS_OK;
}

dtans_status dtans_to_device(dtans_matrix *mat, void *stream) {
    if (!mat) return set_err(DTANS_EINVAL, "null matrix handle");
    return reserve(mat, 1, (hipStream_t)stream);
}

dtans_status dtans_reserve(dtans_matrix *mat, int32_t k, void *stream) {
    if (!mat) return set_err(DTANS_EINVAL, "null matrix handle");
    if (k < 1) return set_err(DTANS_EINVAL, "k must be >= 1");
    return reserve(mat, k, (hipStream_t)stream);
}

dtans_status dtans_set_launch(dtans_matrix *mat, int32_t waves_per_wg, int32_t wg_per_cu,
                              int32_t stream_stage) {
    if (!mat) return set_err(DTANS_EINVAL, "null matrix handle");
    if (waves_per_wg < 0 || waves_per_wg > 16 || wg_per_cu < 0 || wg_per_cu > 32)
        return set_err(DTANS_EINVAL, "waves_per_wg must be 0..16 and wg_per_cu 0..32");
    if (stream_stage < 0 || stream_stage > DTANS_STAGE_RING)
        return set_err(DTANS_EINVAL, "stream_stage must be 0, 1 or 2");
    if (waves_per_wg) mat->waves_per_wg = waves_per_wg;
    if (wg_per_cu) mat->wg_per_cu = wg_per_cu;
    if (stream_stage) mat->stage = stream_stage;
    return DTANS_OK;
}

dtans_status dtans_matrix_info(const dtans_matrix *mat, dtans_info *o) {
    if (!mat || !o) return set_err(DTANS_EINVAL, "null argument");
    const Container &c = mat->c;
    memset(o, 0, sizeof(*o));
    const int64_t vb = (int64_t)c.value_bytes();
    o->m = c.m;
    o->n = c.n;
    o->nnz = c.nnz;
    o->dtype = (int32_t)c.dtype;
    o->layout = (int32_t)c.layout;
    o->lane_nnz = (int32_t)c.lane_nnz;
    o->waves_per_wg = uses_ring(mat) ? plan_launch(mat).ring_waves_per_wg : plan_launch(mat).waves_per_wg;
    o->num_lanes = c.num_lanes;
    o->num_waves = c.num_waves;
    o->words = (int64_t)c.words.size();
    o->esc_delta = (int64_t)c.escd.size();
    o->esc_value = (int64_t)c.escv.size();
    o->table_bytes = (int64_t)kSlots * (8 + vb);
    o->stream_bytes = 4 * o->words + 4 * o->esc_delta + vb * o->esc_value;
    int64_t nsplit = 0;
    if (c.layout == kLayoutNnz) {
        std::vector<int32_t> lr, sr, sf, sl;
        nnz_layout_meta(c, lr, sr, sf, sl);
        nsplit = (int64_t)sr.size();
    }
    // what the kernels read besides tables and streams: row pointers (row
    // layout) or the nonempty-row list and empty rows (nonzero layout), the
    // per-wave offsets, and the lane and split-row lists
    int64_t nonempty = 0;
    for (int64_t i = 0; i < c.m; ++i) nonempty += c.row_ptr[i] < c.row_ptr[i + 1];
    o->index_bytes = 3 * 8 * (c.num_waves + 1) +
                     (c.layout == kLayoutNnz
                          ? 8 * (nonempty + 1) + 4 * (c.m - nonempty) + 4 * c.num_lanes + 12 * nsplit
                          : 4 * (c.m + 1));
    o->total_bytes = o->table_bytes + o->stream_bytes + o->index_bytes;
    o->csr_bytes = 4 * (c.m + 1) + c.nnz * (4 + vb);
    o->coo_bytes = c.nnz * (8 + vb);
    o->sell_bytes = sell_bytes(c, 32);
    o->delta_symbols = c.dtab.symbols;
    o->value_symbols = c.vtab.symbols;
    o->delta_entropy = c.dtab.entropy;
    o->value_entropy = c.vtab.entropy;
    o->delta_cross_entropy = c.dtab.cross_entropy;
    o->value_cross_entropy = c.vtab.cross_entropy;
    o->bits_per_nnz = c.nnz ? 8.0 * o->stream_bytes / c.nnz : 0.0;
    o->stream_stage = uses_ring(mat) ? DTANS_STAGE_RING : DTANS_STAGE_DIRECT;
    o->first_delta_column = c.first_mode == 0;
    o->escape_in_stream = c.esc_mode == 1;
    o->sort_window = (int32_t)c.sigma;
    o->direct_table = 1;
    for (int i = 0; i < kSlots; ++i)
        if (((c.dtab.flags[i] & 1) && c.dtab.base[i] > 255) || ((c.vtab.flags[i] & 1) && c.vtab.base[i] > 255))
            o->direct_table = 0;
    return DTANS_OK;
}

namespace {
// argument checks shared by dtans_spmm and dtans_spmm_noalloc
dtans_status spmm_args(const dtans_matrix *mat, int32_t k, const void *X, int64_t ldx, const void *Y,
                       int64_t ldy) {
    const Container &c = mat->c;
    if (ldx < k || ldy < k) return set_err(DTANS_EINVAL, "leading dimensions must be >= k");
    if (ldx >= (1ll << 31) || ldy >= (1ll << 31)) return set_err(DTANS_ERANGE, "leading dimensions must be below 2^31");
    if ((c.m > 0 && !Y) || (c.n > 0 && c.nnz > 0 && !X)) return set_err(DTANS_EINVAL, "null vector");
    return DTANS_OK;
}
}  // namespace

dtans_status dtans_spmm(dtans_matrix *mat, int32_t k, const void *X, int64_t ldx, void *Y,
                        int64_t ldy, double alpha, double beta, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    if (k < 1) return set_err(DTANS_EINVAL, "k must be >= 1");
    dtans_status s = ready(mat, k);
    if (s) return s;
    s = spmm_args(mat, k, X, ldx, Y, ldy);
    if (s) return s;
    hipError_t e = launch_spmm(mat->view, mat->c.dtype == kF64, k, X, ldx, Y, ldy, alpha, beta,
                               (double *)mat->scratch, plan_launch(mat), st);
    if (e != hipSuccess) return hip_err(e, "dtans_spmm launch");
    return DTANS_OK;
}

dtans_status dtans_spmm_noalloc(dtans_matrix *mat, int32_t k, const void *X, int64_t ldx, void *Y,
                                int64_t ldy, double alpha, double beta, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    if (k < 1) return set_err(DTANS_EINVAL, "k must be >= 1");
    dtans_status s = ready(mat, 0);  // the handle's own scratch is not used
    if (s) return s;
    s = spmm_args(mat, k, X, ldx, Y, ldy);
    if (s) return s;
    const size_t need = spmm_scratch_bytes(mat->view, k);
    if (need > kStaticScratchBytes)
        return set_err(DTANS_ERANGE, "dtans_spmm_noalloc: this product needs " + std::to_string(need) +
                                         " bytes of scratch, above the library's fixed " +
                                         std::to_string(kStaticScratchBytes) +
                                         " bytes; use dtans_spmm after dtans_reserve");
    void *ptr = nullptr;
    hipError_t e = static_scratch(&ptr);
    if (e != hipSuccess) return hip_err(e, "dtans_spmm_noalloc scratch lookup");
    e = launch_spmm(mat->view, mat->c.dtype == kF64, k, X, ldx, Y, ldy, alpha, beta, (double *)ptr,
                    plan_launch(mat), st);
    if (e != hipSuccess) return hip_err(e, "dtans_spmm_noalloc launch");
    return DTANS_OK;
}

dtans_status dtans_spmv(dtans_matrix *mat, const void *x, void *y, double alpha, double beta,
                        void *stream) {
    return dtans_spmm(mat, 1, x, 1, y, 1, alpha, beta, stream);
}

dtans_status dtans_spmm_t(dtans_matrix *mat, int32_t k, const void *dY, int64_t lddy, void *dX,
                          int64_t lddx, double alpha, double beta, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    if (k < 1) return set_err(DTANS_EINVAL, "k must be >= 1");
    // the per-CU blocks of dX live in the handle's scratch (see launch_spmm_t)
    dtans_status s = ready(mat, 1);
    if (s) return s;
    const Container &c = mat->c;
    if (lddy < k || lddx < k) return set_err(DTANS_EINVAL, "leading dimensions must be >= k");
    if (lddx >= (1ll << 31) || lddy >= (1ll << 31)) return set_err(DTANS_ERANGE, "leading dimensions must be below 2^31");
    if ((c.n > 0 && !dX) || (c.m > 0 && c.nnz > 0 && !dY)) return set_err(DTANS_EINVAL, "null vector");
    hipError_t e = launch_spmm_t(mat->view, c.dtype == kF64, k, dY, lddy, dX, lddx, alpha, beta,
                                 plan_launch(mat), mat->scratch, mat->scratch_bytes, st);
    if (e != hipSuccess) return hip_err(e, "dtans_spmm_t launch");
    return DTANS_OK;
}

dtans_status dtans_spmv_sym(dtans_matrix *mat, const void *diag, const void *x, void *y, double alpha,
                            double beta, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    dtans_status s = ready(mat, 1);
    if (s) return s;
    const Container &c = mat->c;
    if (c.m != c.n) return set_err(DTANS_EINVAL, "the triangle of a symmetric matrix must be square");
    if (c.sigma) return set_err(DTANS_EUNSUPPORTED, "the symmetric product needs rows in CSR order");
    if (c.m > 0 && (!x || !y)) return set_err(DTANS_EINVAL, "null vector");
    if (x == y && c.m > 0) return set_err(DTANS_EINVAL, "y must not alias x");
    // sums = beta y + alpha d .* x, then sums += alpha (S + S^T) x, in FP64: y
    // itself, or the handle's scratch and rounded once into y
    const bool f64 = c.dtype == kF64;
    double *sums = f64 ? (double *)y : sym_sums_bytes(c) ? (double *)mat->scratch : nullptr;
    hipError_t e = launch_sym_start(f64, diag, x, y, sums, c.m, alpha, beta, st);
    if (e != hipSuccess) return hip_err(e, "dtans_spmv_sym start launch");
    if (!sums) return DTANS_OK;  // no nonzeros
    e = launch_sym(mat->view, f64, x, sums, alpha, plan_launch(mat), st);
    if (e != hipSuccess) return hip_err(e, "dtans_spmv_sym launch");
    if (!f64) e = launch_sym_end(sums, (float *)y, c.m, st);
    if (e != hipSuccess) return hip_err(e, "dtans_spmv_sym end launch");
    return DTANS_OK;
}

dtans_status dtans_decode_csr(dtans_matrix *mat, int32_t *row_ptr, int32_t *col_idx, void *vals,
                              void *stream) {
    hipStream_t st = (hipStream_t)stream;
    dtans_status s = ready(mat, 0);
    if (s) return s;
    const Container &c = mat->c;
    if (!row_ptr || (c.nnz > 0 && (!col_idx || !vals))) return set_err(DTANS_EINVAL, "null output");
    // the original matrix (row-sorted containers decode into its positions)
    HIP_TRY(hipMemcpyAsync(row_ptr, c.sigma ? mat->view.orig_row_ptr : mat->view.row_ptr, 4 * (size_t)(c.m + 1),
                           hipMemcpyDeviceToDevice, st));
    hipError_t e = launch_decode(mat->view, c.dtype == kF64, col_idx, vals, plan_launch(mat), st);
    if (e != hipSuccess) return hip_err(e, "dtans_decode_csr launch");
    return DTANS_OK;
}

void dtans_destroy(dtans_matrix *mat) {
    if (!mat) return;
    if (mat->scratch && !mat->scratch_in_bufs) (void)hipFree(mat->scratch);
    delete mat;
}

// ------------------------------------------------------------------ batch
dtans_status dtans_batch_create(int32_t count, dtans_matrix *const *mats, dtans_batch **out) {
    if (!out || !mats || count <= 0) return set_err(DTANS_EINVAL, "need at least one matrix");
    *out = nullptr;
    if (count > kMaxBatch) return set_err(DTANS_EINVAL, "at most 128 matrices per batch");
    const bool f64 = mats[0] && mats[0]->c.dtype == kF64;
    for (int i = 0; i < count; ++i) {
        if (!mats[i]) return set_err(DTANS_EINVAL, "null matrix in batch");
        if ((mats[i]->c.dtype == kF64) != f64) return set_err(DTANS_EINVAL, "batch matrices must share a dtype");
        if (mats[i]->c.layout != kLayoutRow)
            return set_err(DTANS_EUNSUPPORTED, "batch matrices must use the ROW layout");
        if (mats[i]->c.n * (int64_t)mats[i]->c.value_bytes() > (1ll << 32))
            return set_err(DTANS_EUNSUPPORTED, "batch matrices must have x of at most 4 GiB");
        dtans_status s = reserve(mats[i], 1, nullptr);
        if (s) return s;
        if (mats[i]->device != mats[0]->device) return set_err(DTANS_EINVAL, "batch matrices on different devices");
    }
    dtans_batch *b = new dtans_batch();
    b->mats.assign(mats, mats + count);
    b->f64 = f64;
    // cost of each encoded wave: its stream words plus a fixed per-wave cost
    std::vector<int32_t> wmat;
    std::vector<int32_t> wid;
    std::vector<double> cost;
    for (int i = 0; i < count; ++i) {
        const Container &c = mats[i]->c;
        for (int64_t w = 0; w < c.num_waves; ++w) {
            wmat.push_back(i);
            wid.push_back((int32_t)w);
            cost.push_back((double)(c.word_off[w + 1] - c.word_off[w]) + 256.0);
        }
    }
    int wpw = 0, wgcu = 0;
    default_shape(f64, 7, wpw, wgcu);  // batch_kernel allows 7 waves per SIMD
    const int64_t total_waves = (int64_t)wmat.size();
    int grid = (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)mats[0]->num_cus * wgcu,
                                                           (total_waves + wpw - 1) / wpw));
    // contiguous ranges of about equal cost, one per workgroup, each split
    // into per-matrix tasks (measured: cutting the ranges at matrix
    // boundaries instead, so that no workgroup restages its tables, is
    // slower)
    std::vector<double> prefix(total_waves + 1, 0.0);
    for (int64_t i = 0; i < total_waves; ++i) prefix[i + 1] = prefix[i] + cost[i];
    b->wg_task.push_back(0);
    int64_t w = 0;
    for (int g = 0; g < grid; ++g) {
        const double goal = prefix[total_waves] * (g + 1) / grid;
        int64_t end = g == grid - 1 ? total_waves
                                    : std::lower_bound(prefix.begin(), prefix.end(), goal) - prefix.begin();
        end = std::max(w, std::min(end, total_waves));
        for (int64_t q = w; q < end;) {
            int64_t e = q;
            while (e < end && wmat[e] == wmat[q]) ++e;
            b->tasks.push_back({wmat[q], wid[q], (int32_t)(e - q), 0});
            q = e;
        }
        b->wg_task.push_back((int32_t)b->tasks.size());
        w = end;
    }
    std::vector<DevMat> views(count);
    for (int i = 0; i < count; ++i) views[i] = mats[i]->view;
    void *p_mats, *p_tasks, *p_wg, *p_ptrs;
    hipStream_t st = nullptr;
    hipError_t e;
    if ((e = b->bufs.upload(&p_mats, views.data(), sizeof(DevMat) * views.size(), st)) != hipSuccess ||
        (e = b->bufs.upload(&p_tasks, b->tasks.data(), sizeof(BatchTask) * b->tasks.size(), st)) != hipSuccess ||
        (e = b->bufs.upload(&p_wg, b->wg_task.data(), 4 * b->wg_task.size(), st)) != hipSuccess ||
        (e = b->bufs.upload(&p_ptrs, nullptr, 2 * sizeof(void *) * (size_t)count, st)) != hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess) {
        delete b;
        return hip_err(e, "dtans_batch_create upload");
    }
    b->dev.mats = (const DevMat *)p_mats;
    b->dev.tasks = (const BatchTask *)p_tasks;
    b->dev.wg_task = (const int32_t *)p_wg;
    b->dev.ptrs = (void *const *)p_ptrs;
    b->launch.waves_per_wg = wpw;
    b->launch.grid = grid;
    *out = b;
    return DTANS_OK;
}

dtans_status dtans_batch_spmv(dtans_batch *b, const void *const *xs, void *const *ys, double alpha,
                              double beta, void *stream) {
    if (!b || !xs || !ys) return set_err(DTANS_EINVAL, "null argument");
    hipStream_t st = (hipStream_t)stream;
    const size_t cnt = b->mats.size();
    BatchPtrs ptrs{};
    for (size_t i = 0; i < cnt; ++i) {
        if ((b->mats[i]->c.m > 0 && !ys[i]) || (b->mats[i]->c.nnz > 0 && !xs[i]))
            return set_err(DTANS_EINVAL, "null vector in batch");
        ptrs.xs[i] = xs[i];
        ptrs.ys[i] = ys[i];
    }
    hipError_t e = launch_batch(b->dev, ptrs, (int)cnt, b->f64, alpha, beta, b->launch, st);
    if (e != hipSuccess) return hip_err(e, "dtans_batch_spmv launch");
    return DTANS_OK;
}

dtans_status dtans_batch_spmm(dtans_batch *b, int32_t k, const void *const *Xs, void *const *Ys, double alpha,
                              double beta, void *stream) {
    if (!b || !Xs || !Ys) return set_err(DTANS_EINVAL, "null argument");
    if (k < 1) return set_err(DTANS_EINVAL, "k must be at least 1");
    hipStream_t st = (hipStream_t)stream;
    const size_t cnt = b->mats.size();
    const size_t vb = b->f64 ? 8 : 4;
    BatchPtrs ptrs{};
    bool aligned = (k * vb) % 16 == 0;
    for (size_t i = 0; i < cnt; ++i) {
        const Container &c = b->mats[i]->c;
        if ((c.m > 0 && !Ys[i]) || (c.nnz > 0 && !Xs[i])) return set_err(DTANS_EINVAL, "null matrix in batch");
        if (c.n * (int64_t)k * (int64_t)vb > (1ll << 32)) aligned = false;  // 32-bit byte offsets
        if ((uintptr_t)Xs[i] % 16 || (uintptr_t)Ys[i] % 16) aligned = false;
        ptrs.xs[i] = Xs[i];
        ptrs.ys[i] = Ys[i];
    }
    hipError_t e = launch_batch_spmm(b->dev, ptrs, (int)cnt, b->f64, k, aligned, alpha, beta, b->launch, st);
    if (e != hipSuccess) return hip_err(e, "dtans_batch_spmm launch");
    return DTANS_OK;
}

void dtans_batch_destroy(dtans_batch *b) { delete b; }

// -------------------------------------------------------------- CSR baseline
dtans_status dtans_csr_create(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr,
                              const int32_t *col_idx, const void *vals, dtans_dtype dtype,
                              int32_t variant, dtans_csr **out) {
    if (!out) return set_err(DTANS_EINVAL, "out is null");
    *out = nullptr;
    if (m < 0 || n < 0 || nnz < 0 || !row_ptr || (nnz > 0 && (!col_idx || !vals)))
        return set_err(DTANS_EINVAL, "bad CSR arguments");
    if (dtype != DTANS_F32 && dtype != DTANS_F64) return set_err(DTANS_EINVAL, "bad dtype");
    if (m >= (1ll << 31) || n >= (1ll << 31) || nnz >= (1ll << 31)) return set_err(DTANS_ERANGE, "sizes must be below 2^31");
    if (row_ptr[0] != 0 || row_ptr[m] != nnz) return set_err(DTANS_EINVAL, "row_ptr must run from 0 to nnz");
    int64_t maxlen = 0;
    for (int64_t i = 0; i < m; ++i) {
        if (row_ptr[i + 1] < row_ptr[i]) return set_err(DTANS_EINVAL, "row_ptr decreases");
        maxlen = std::max<int64_t>(maxlen, row_ptr[i + 1] - row_ptr[i]);
    }
    for (int64_t q = 0; q < nnz; ++q)
        if (col_idx[q] < 0 || col_idx[q] >= n) return set_err(DTANS_ERANGE, "column index out of range");
    const double mean = m ? (double)nnz / m : 0.0;
    if (variant == 0) variant = 3;
    if (variant < 1 || variant > 3) return set_err(DTANS_EINVAL, "variant must be 0, 1, 2 or 3");
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    dtans_csr *h = new dtans_csr();
    h->m = m;
    h->n = n;
    h->nnz = nnz;
    h->f64 = dtype == DTANS_F64;
    h->device = dev;
    h->num_cus = device_cus(dev);
    const size_t vb = h->f64 ? 8 : 4;
    CsrDev &c = h->dev;
    c.m = m;
    c.n = n;
    c.nnz = nnz;
    c.variant = variant;
    int G = 1;
    while (G < 64 && G < mean) G <<= 1;
    c.group = G;
    c.lane_nnz = 32;
    std::vector<int32_t> lane_row, split_row, split_first, split_last, split_long;
    if (variant == 2) {
        Container tmp;  // only row_ptr and the lane geometry are used
        tmp.layout = kLayoutNnz;
        tmp.lane_nnz = (uint32_t)c.lane_nnz;
        tmp.m = m;
        tmp.nnz = nnz;
        tmp.num_lanes = (nnz + c.lane_nnz - 1) / c.lane_nnz;
        tmp.row_ptr.assign(row_ptr, row_ptr + m + 1);
        nnz_layout_meta(tmp, lane_row, split_row, split_first, split_last);
        c.num_lanes = tmp.num_lanes;
        split_long = long_splits(split_first, split_last, kLongSplit);
    }
    std::vector<int32_t> blk;  // CSR-stream row blocks: <= 1024 nonzeros or one long row
    if (variant == 3) {
        const int64_t cap = 1024, max_rows = 4096;
        blk.push_back(0);
        int64_t r = 0;
        while (r < m) {
            int64_t e = r, cnt = 0;
            while (e < m && e - r < max_rows && cnt + (row_ptr[e + 1] - row_ptr[e]) <= cap) {
                cnt += row_ptr[e + 1] - row_ptr[e];
                ++e;
            }
            if (e == r) e = r + 1;  // a row longer than the block: its own block
            blk.push_back((int32_t)e);
            r = e;
        }
        c.nblk = (int64_t)blk.size() - 1;
    }
    void *p[9];
    hipStream_t st = nullptr;
    hipError_t e;
    if ((e = h->bufs.upload(&p[7], blk.data(), 4 * blk.size(), st)) != hipSuccess ||
        (e = h->bufs.upload(&p[0], row_ptr, 4 * (size_t)(m + 1), st)) != hipSuccess ||
        (e = h->bufs.upload(&p[1], col_idx, 4 * (size_t)nnz, st)) != hipSuccess ||
        (e = h->bufs.upload(&p[2], vals, vb * (size_t)nnz, st)) != hipSuccess ||
        (e = h->bufs.upload(&p[3], lane_row.data(), 4 * lane_row.size(), st)) != hipSuccess ||
        (e = h->bufs.upload(&p[4], split_row.data(), 4 * split_row.size(), st)) != hipSuccess ||
        (e = h->bufs.upload(&p[5], split_first.data(), 4 * split_first.size(), st)) != hipSuccess ||
        (e = h->bufs.upload(&p[6], split_last.data(), 4 * split_last.size(), st)) != hipSuccess ||
        (e = h->bufs.upload(&p[8], split_long.data(), 4 * split_long.size(), st)) != hipSuccess ||
        (variant == 2 && (e = h->bufs.upload((void **)&h->partial, nullptr,
                                             sizeof(double) * (size_t)(2 * c.num_lanes * kMaxPassCols + 1),
                                             st)) != hipSuccess) ||
        (e = hipStreamSynchronize(st)) != hipSuccess) {
        delete h;
        return hip_err(e, "dtans_csr_create upload");
    }
    c.row_ptr = (const int32_t *)p[0];
    c.col = (const int32_t *)p[1];
    c.val = p[2];
    c.lane_row = (const int32_t *)p[3];
    c.split.row = (const int32_t *)p[4];
    c.split.first = (const int32_t *)p[5];
    c.split.last = (const int32_t *)p[6];
    c.split.longs = (const int32_t *)p[8];
    c.split.n = (int64_t)split_row.size();
    c.split.n_long = (int64_t)split_long.size();
    c.blk = (const int32_t *)p[7];
    h->bytes = 4 * (m + 1) + nnz * (4 + (int64_t)vb) +
               (variant == 2 ? 4 * c.num_lanes + 12 * c.split.n : 0) +
               (variant == 3 ? 4 * (c.nblk + 1) : 0);
    *out = h;
    return DTANS_OK;
}

dtans_status dtans_csr_spmm(dtans_csr *h, int32_t k, const void *X, int64_t ldx, void *Y,
                            int64_t ldy, double alpha, double beta, void *stream) {
    if (!h) return set_err(DTANS_EINVAL, "null CSR handle");
    if (k < 1 || ldx < k || ldy < k) return set_err(DTANS_EINVAL, "bad k or leading dimension");
    if ((h->m > 0 && !Y) || (h->nnz > 0 && !X)) return set_err(DTANS_EINVAL, "null vector");
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != h->device) return set_err(DTANS_EINVAL, "CSR handle lives on another device");
    hipError_t e = launch_csr(h->dev, h->f64, k, X, ldx, Y, ldy, alpha, beta, h->partial, h->num_cus,
                              (hipStream_t)stream);
    if (e != hipSuccess) return hip_err(e, "dtans_csr_spmm launch");
    return DTANS_OK;
}

dtans_status dtans_csr_spmv(dtans_csr *h, const void *x, void *y, double alpha, double beta,
                            void *stream) {
    return dtans_csr_spmm(h, 1, x, 1, y, 1, alpha, beta, stream);
}

int64_t dtans_csr_bytes(const dtans_csr *h) { return h ? h->bytes : 0; }

void dtans_csr_destroy(dtans_csr *h) {
    delete h;
}

int32_t dtans_autotune_candidates(int64_t m, int64_t nnz, const int32_t *row_ptr,
                                  dtans_dtype dtype, int32_t k, const dtans_encode_opts *in,
                                  dtans_encode_opts *out, int32_t cap) {
    std::vector<dtans_encode_opts> c;
    if (cap < 0 || (cap > 0 && !out)) {
        set_err(DTANS_EINVAL, "out must hold cap >= 0 entries");
        return -1;
    }
    if (tune_candidates(m, nnz, row_ptr, dtype, k, in, c) != DTANS_OK) return -1;
    for (int32_t i = 0; i < cap && i < (int32_t)c.size(); ++i) out[i] = c[i];
    return (int32_t)c.size();
}

dtans_status dtans_autotune(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr,
                            const int32_t *col_idx, const void *vals, dtans_dtype dtype, int32_t k,
                            double budget_s, const char *cache_path, dtans_encode_opts *inout,
                            double *best_ms) {
    const auto t_start = std::chrono::steady_clock::now();
    if (!inout) return set_err(DTANS_EINVAL, "inout is null");
    if (!(budget_s >= 0)) return set_err(DTANS_EINVAL, "budget_s must be >= 0");
    if (n < 0 || n >= (1ll << 31)) return set_err(DTANS_ERANGE, "columns must be 0..2^31-1");
    if (nnz > 0 && (!col_idx || !vals)) return set_err(DTANS_EINVAL, "null array");
    std::vector<dtans_encode_opts> cands;
    dtans_status s = tune_candidates(m, nnz, row_ptr, dtype, k, inout, cands);
    if (s) return s;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, dev));
    std::string devname = std::string(prop.name) + "/" + prop.gcnArchName;
    for (char &ch : devname)
        if (ch == ' ' || ch == '\t' || ch == '\n') ch = '_';

    // fingerprint of the problem: sizes, dtype, k, the fixed options, the
    // arrays, and a number raised when the kernels' relative speeds change, so
    // that results of earlier kernels are not taken from the cache
    constexpr uint64_t kKernelSet = 2;
    Fingerprint fp;
    fp.word(kKernelSet);
    for (int64_t w : {m, n, nnz, (int64_t)dtype, (int64_t)k, (int64_t)inout->layout,
                      (int64_t)inout->lane_nnz, (int64_t)inout->waves_per_wg,
                      (int64_t)inout->wg_per_cu, (int64_t)inout->sort_rows,
                      (int64_t)inout->stream_stage, (int64_t)inout->max_mult})
        fp.word((uint64_t)w);
    fp.word(inout->perm_seed);
    if (cache_path) {
        fp.bytes(row_ptr, 4 * (size_t)(m + 1));
        if (nnz > 0) {
            fp.bytes(col_idx, 4 * (size_t)nnz);
            fp.bytes(vals, (dtype == DTANS_F64 ? 8 : 4) * (size_t)nnz);
        }
        char key[17];
        snprintf(key, sizeof key, "%016llx", (unsigned long long)fp.h);
        if (FILE *f = fopen(cache_path, "r")) {
            char line[1024];
            while (fgets(line, sizeof line, f)) {
                char tag[32], fk[32], dn[512];
                int lay, T, w, g, st;
                double ms;
                if (sscanf(line, "%31s %31s %511s %d %d %d %d %d %lf", tag, fk, dn, &lay, &T, &w, &g,
                           &st, &ms) == 9 &&
                    strcmp(tag, "dtans-autotune-v2") == 0 && strcmp(fk, key) == 0 && devname == dn) {
                    fclose(f);
                    inout->layout = lay;
                    inout->lane_nnz = T;
                    inout->waves_per_wg = w;
                    inout->wg_per_cu = g;
                    inout->stream_stage = st;
                    if (best_ms) *best_ms = ms;
                    return DTANS_OK;
                }
            }
            fclose(f);
        }
    }

    TuneResources r;
    HIP_TRY(hipStreamCreate(&r.st));
    const size_t vb = dtype == DTANS_F64 ? 8 : 4;
    void *X = nullptr, *Y = nullptr, *flush = nullptr;
    HIP_TRY(r.bufs.upload(&X, nullptr, (size_t)std::max<int64_t>(n, 1) * k * vb, r.st));
    HIP_TRY(r.bufs.upload(&Y, nullptr, (size_t)std::max<int64_t>(m, 1) * k * vb, r.st));
    // x = 0x3f3f... bit patterns: finite, nonzero values of either width
    HIP_TRY(hipMemsetAsync(X, 0x3f, (size_t)std::max<int64_t>(n, 1) * k * vb, r.st));
    const int64_t flush_bytes = 512ll << 20;
    HIP_TRY(r.bufs.upload(&flush, nullptr, flush_bytes, r.st));
    uint32_t *sink = (uint32_t *)((char *)flush + flush_bytes);  // inside the 256-byte pad
    const int kMaxReps = 25;
    r.ev.resize(2 * kMaxReps);
    for (auto &e : r.ev) HIP_TRY(hipEventCreate(&e));

    double best = INFINITY;
    dtans_encode_opts best_o = cands[0];
    size_t i = 0;
    while (i < cands.size()) {
        double elapsed = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
        if (i > 0 && elapsed > budget_s) break;
        // encode once for every launch shape of this encoding
        dtans_encode_opts eo = cands[i];
        eo.waves_per_wg = 0;
        eo.wg_per_cu = 0;
        if (r.h) {
            dtans_destroy(r.h);
            r.h = nullptr;
        }
        s = dtans_encode_csr(m, n, nnz, row_ptr, col_idx, vals, dtype, &eo, &r.h);
        if (s) return s;
        s = dtans_reserve(r.h, k, r.st);
        if (s) return s;
        size_t j = i;
        for (; j < cands.size() && cands[j].layout == cands[i].layout &&
               cands[j].lane_nnz == cands[i].lane_nnz;
             ++j) {
            s = dtans_set_launch(r.h, cands[j].waves_per_wg, cands[j].wg_per_cu,
                                 cands[j].stream_stage);
            if (s) return s;
            auto run = [&]() { return dtans_spmm(r.h, k, X, k, Y, k, 1.0, 0.0, r.st); };
            // two untimed launches, then one timed to size the repetitions
            for (int w = 0; w < 2; ++w)
                if ((s = run())) return s;
            HIP_TRY(launch_flush(flush, flush_bytes, sink, r.st));
            HIP_TRY(hipEventRecord(r.ev[0], r.st));
            if ((s = run())) return s;
            HIP_TRY(hipEventRecord(r.ev[1], r.st));
            HIP_TRY(hipEventSynchronize(r.ev[1]));
            float probe = 0;
            HIP_TRY(hipEventElapsedTime(&probe, r.ev[0], r.ev[1]));
            // about 0.1 s of launches per shape (each rep also reads the flush buffer)
            const int reps = (int)std::min<double>(kMaxReps, std::max(3.0, 100.0 / (probe + 0.15)));
            for (int q = 0; q < reps; ++q) {
                HIP_TRY(launch_flush(flush, flush_bytes, sink, r.st));
                HIP_TRY(hipEventRecord(r.ev[2 * q], r.st));
                if ((s = run())) return s;
                HIP_TRY(hipEventRecord(r.ev[2 * q + 1], r.st));
            }
            HIP_TRY(hipStreamSynchronize(r.st));
            std::vector<float> t(reps);
            for (int q = 0; q < reps; ++q) HIP_TRY(hipEventElapsedTime(&t[q], r.ev[2 * q], r.ev[2 * q + 1]));
            std::sort(t.begin(), t.end());
            const double med = t[reps / 2];
            if (med < best) {
                best = med;
                best_o = cands[j];
            }
        }
        i = j;
    }
    inout->layout = best_o.layout;
    inout->lane_nnz = best_o.lane_nnz;
    inout->waves_per_wg = best_o.waves_per_wg;
    inout->wg_per_cu = best_o.wg_per_cu;
    inout->stream_stage = best_o.stream_stage;
    if (best_ms) *best_ms = best;
    if (cache_path) {
        FILE *f = fopen(cache_path, "a");
        if (!f) return set_err(DTANS_EIO, std::string("cannot append to ") + cache_path);
        int ok = fprintf(f, "dtans-autotune-v2 %016llx %s %d %d %d %d %d %.6f\n",
                         (unsigned long long)fp.h, devname.c_str(), best_o.layout, best_o.lane_nnz,
                         best_o.waves_per_wg, best_o.wg_per_cu, best_o.stream_stage, best);
        if (fclose(f) != 0 || ok < 0) return set_err(DTANS_EIO, std::string("cannot write ") + cache_path);
    }
    return DTANS_OK;
}

}  // extern "C"
