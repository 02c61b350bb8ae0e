// C ABI entry points: dataset handles, argument checking, profiling, error text.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <exception>
#include <mutex>
#include <new>
#include <thread>

#include "common.h"
#include "grid_sync.h"
#include "host_util.h"

namespace tron {

Tuning g_tuning;

// ------------------------------------------------------------------ errors
static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

int hip_fail(hipError_t e, const char *what, const char *file, int line)
{
    const char *base = strrchr(file, '/');
    set_error("HIP error %d (%s) in %s at %s:%d", (int)e, hipGetErrorString(e), what, base ? base + 1 : file, line);
    return (e == hipErrorOutOfMemory) ? TRON_ENOMEM : TRON_EDEVICE;
}

// ------------------------------------------------------------------ profiler
const char *const kSlotNames[SLOT_COUNT] = {
    "spmv_fwd", "spmv_bwd", "spmv_head", "spmv_tiles", "spmv_tile_reduce", "spmv_gather", "spmv_fixup", "spmv_combine", "loss_terms",
    "dense_fun_grad", "dense_hv", "dense_finalize", "dense_compact", "dot", "reduce_final", "cg_vec", "batch_pass", "batch_advance"};

int Profiler::begin(int slot, hipStream_t st)
{
    if (used == pool.size()) {
        Rec r;
        if (hipEventCreate(&r.a) != hipSuccess) return -1;
        if (hipEventCreate(&r.b) != hipSuccess) { hipEventDestroy(r.a); return -1; }
        r.slot = slot;
        pool.push_back(r);
    }
    Rec &r = pool[used];
    r.slot = slot;
    if (hipEventRecord(r.a, st) != hipSuccess) return -1;
    return (int)used++;
}

void Profiler::end(int idx, hipStream_t st) { hipEventRecord(pool[idx].b, st); }

int Profiler::drain()
{
    for (size_t i = 0; i < used; ++i) {
        Rec &r = pool[i];
        TRON_HIP(hipEventSynchronize(r.b));
        float t = 0.f;
        TRON_HIP(hipEventElapsedTime(&t, r.a, r.b));
        ms[r.slot] += t;
        calls[r.slot] += 1;
    }
    used = 0;
    return TRON_OK;
}

void Profiler::destroy()
{
    for (auto &r : pool) { hipEventDestroy(r.a); hipEventDestroy(r.b); }
    pool.clear();
    used = 0;
}

// ------------------------------------------------------------------ helpers
static int check_device()
{
    int count = 0;
    hipError_t e = hipGetDeviceCount(&count);
    if (e != hipSuccess || count < 1) {
        set_error("no usable HIP device (%s); this library has no CPU fallback", hipGetErrorString(e));
        (void)hipGetLastError();
        return TRON_EDEVICE;
    }
    return TRON_OK;
}

static int alloc_common(tron_dataset *ds)
{
    const int64_t n = ds->n;
    TRON_HIP(hipGetDevice(&ds->device));
    if (ds->dense) TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->y8), (size_t)n));
    else TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->y), sizeof(double) * n));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->Dbuf[0]), sizeof(double) * n));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->Dbuf[1]), sizeof(double) * n));
    if (!ds->dense) {
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->z), sizeof(double) * n));
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->zhat), sizeof(double) * n));
    }
    int64_t need = 4 * (int64_t)kMaxGrid;
    if (ds->dense) {
        ds->dense_grid = dense_grid_for(ds->n, ds->d);
        const int64_t dn = dense_partials_needed(ds->n, ds->d);
        if (dn > need) need = dn;
    }
    ds->partials_len = need;
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->partials), sizeof(double) * need));
    // The scalars the host steers by live in pinned host memory that the kernels write directly: they are there when
    // the stream has drained, without a copy operation between the last kernel and the host's wait.
    TRON_HIP(hipHostMalloc(reinterpret_cast<void **>(&ds->scal_host), sizeof(double) * kHostWords + (ds->dense ? 0 : kSolveHostBytes), hipHostMallocMapped));
    memset(ds->scal_host, 0, sizeof(double) * kHostWords);
    TRON_HIP(hipHostGetDevicePointer(reinterpret_cast<void **>(&ds->scal_dev), ds->scal_host, 0));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->scal_copy), sizeof(double) * kScalars));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->ticket), 64));
    TRON_HIP(hipMemset(ds->ticket, 0, 64));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->sync_words), sizeof(unsigned) * kSyncWords));
    TRON_HIP(hipMemset(ds->sync_words, 0, sizeof(unsigned) * kSyncWords));
    TRON_HIP(hipDeviceGetAttribute(&ds->device_cus, hipDeviceAttributeMultiprocessorCount, ds->device));
    // a stream may be confined to a part of them (hipExtStreamCreateWithCUMask)
    uint32_t mask[32] = {0};
    int masked = 0;
    if (hipExtStreamGetCUMask(ds->stream, 32, mask) != hipSuccess) (void)hipGetLastError();
    for (uint32_t m : mask) masked += __builtin_popcount(m);
    ds->cus = masked > 0 ? std::min(masked, ds->device_cus) : ds->device_cus;
    return TRON_OK;
}

// ------------------------------------------------------------------ launches whose workgroups wait for each other
// 100 ms: far longer than the workgroups of a pass over the largest matrix are apart, and what a solve loses when another process
// holds a part of the GPU
constexpr long long kResidentWaitUs = 100'000, kTicksPerUs = 100;

GridSync grid_sync(const tron_dataset *ds)
{
    const long long us = g_tuning.solve_wait_us;
    return GridSync{ds->sync_words, us < 0 ? kResidentWaitUs * kTicksPerUs : us == 0 ? -1 : us * kTicksPerUs};
}

bool resident_possible(const tron_dataset *ds, int grid) { return g_tuning.solve_resident != 0 && grid <= ds->cus; }

namespace {
struct ResidentPool {
    std::mutex m;
    std::condition_variable freed;
    int wanted = 0;   // workgroups of the solves under way, whatever their way, and of those that wait for room
    int used = 0;     // those of the launches whose workgroups wait for each other
};
constexpr int kPools = 64;
// Several times what the longest solves in one launch take at a loose tolerance: those that take turns get theirs.  One that holds its room for
// longer may have it for a launch that waits behind other work on its stream, for however long that takes.
constexpr std::chrono::milliseconds kRoomWait{10};
ResidentPool g_resident[kPools];
}  // namespace

ResidentShare::ResidentShare(const tron_dataset *ds, int grid, int turns)
    : device_(ds->device), grid_(ds->cus < ds->device_cus ? ds->device_cus : grid)
{
    ResidentPool &p = g_resident[device_ % kPools];
    std::unique_lock<std::mutex> lock(p.m);
    p.wanted += grid_;
    granted_ = turns > 0 && g_tuning.solve_resident < 0 && (2 * grid_ <= ds->device_cus || p.wanted <= turns * ds->device_cus);
    if (!granted_) return;
    granted_ = p.freed.wait_for(lock, kRoomWait, [&] { return p.used == 0 || p.used + grid_ <= ds->device_cus; });
    if (granted_) p.used += grid_;
}

void ResidentShare::give_back()
{
    if (!granted_) return;
    ResidentPool &p = g_resident[device_ % kPools];
    {
        std::lock_guard<std::mutex> lock(p.m);
        p.used -= grid_;
    }
    granted_ = false;
    p.freed.notify_all();
}

ResidentShare::~ResidentShare()
{
    give_back();
    ResidentPool &p = g_resident[device_ % kPools];
    std::lock_guard<std::mutex> lock(p.m);
    p.wanted -= grid_;
}

static int check_labels(const double *y, int64_t n)
{
    for (int64_t i = 0; i < n; ++i)
        if (!(y[i] == 1.0 || y[i] == -1.0)) {
            set_error("y[%lld] = %g is not +1 or -1", (long long)i, y[i]);
            return TRON_EINVAL;
        }
    return TRON_OK;
}

// host copy of a caller's array in device memory
template <typename T>
static int fetch(std::vector<T> &dst, const T *src, size_t count)
{
    try {
        dst.resize(count);
    } catch (const std::bad_alloc &) {
        set_error("out of host memory staging %zu elements", count);
        return TRON_ENOMEM;
    }
    if (count) TRON_HIP(hipMemcpy(dst.data(), src, sizeof(T) * count, hipMemcpyDeviceToHost));
    return TRON_OK;
}

// csr_plan_build for either thread: running out of host memory is an error code
static int plan_build(CsrPlan &P, int64_t rows, int64_t cols, const int64_t *rowptr, const int32_t *col, const double *val, int parts, bool hot,
                      bool unit, int64_t cols_used, hipStream_t st, const CsrFill *fill = nullptr, HostStage *stage = nullptr)
{
    try {
        return csr_plan_build(P, rows, cols, rowptr, col, val, parts, hot, unit, cols_used, st, fill, stage);
    } catch (const std::bad_alloc &) {
        set_error("out of host memory building the sparse layout");
        return TRON_ENOMEM;
    }
}

static int alloc_row_partials(tron_dataset *ds)
{
    int64_t need = 0;
    if (!ds->fwd.plain && !ds->fwd.direct) need = std::max<int64_t>(need, ds->fwd.nseg_total);   // one partial sum per segment
    if (!ds->bwd.plain && !ds->bwd.direct) need = std::max<int64_t>(need, ds->bwd.nseg_total);
    if (need > 0) TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->row_partials), sizeof(double) * need));
    return TRON_OK;
}

// The layouts of a handle of an unpartitioned matrix, built on the device.  rowptr and y are on the host and have been checked.
static int layouts_on_device(tron_dataset *ds, const int64_t *h_rowptr, const int32_t *col, const double *val, const double *h_y, int mem, int64_t rows_used)
{
    const int64_t n = ds->n, d = ds->d, nnz = h_rowptr[n];
    struct Build : CsrDeviceBuild { ~Build() { release(); } } B;
    HostStage stage(ds->stream);   // given back first: it waits for the stream
    TRON_TRY(B.begin(n, d, nnz, h_rowptr, col, val, mem, stage, ds->stream));
    TRON_TRY(stage.copy(ds->y, h_y, sizeof(double) * (size_t)n, ds->stream));
    const CsrFill by_row = B.by_row(), by_column = B.by_column();
    // beside the copies and the sort; what it copies of entries that turn out to be wrong is not used
    TRON_TRY(plan_build(ds->fwd, n, d, h_rowptr, nullptr, nullptr, 1, false, false, 0, ds->stream, &by_row, &stage));
    TRON_TRY(B.wait());
    if (*B.bad != ~0ull) {   // the first in row order
        const int64_t k = (int64_t)*B.bad, row = std::upper_bound(h_rowptr, h_rowptr + n + 1, k) - h_rowptr - 1;
        int32_t c[2] = {-1, -1};   // the entry's column and the one before in its row
        for (int j = 0; j < 2; ++j)
            if (k - j >= h_rowptr[row]) TRON_HIP(hipMemcpy(&c[j], B.col + k - j, sizeof(int32_t), hipMemcpyDeviceToHost));
        if (c[0] <= c[1] || c[0] >= d || c[0] < 0)
            set_error("row %lld: column index %lld out of order or out of range [0,%lld)", (long long)row, (long long)c[0], (long long)d);
        else set_error("row %lld: non-finite value", (long long)row);
        return TRON_EINVAL;
    }
    int64_t cols_used = 0;
    for (int64_t j = 0; j < d; ++j) cols_used += B.t_rowptr[j + 1] > B.t_rowptr[j];
    if (!ds->fwd.plain) ds->fwd.cold_cols = cols_used;
    TRON_TRY(plan_build(ds->bwd, d, n, B.t_rowptr, nullptr, nullptr, 1, false, false, rows_used, ds->stream, &by_column, &stage));
    TRON_HIP(hipStreamSynchronize(ds->stream));   // what went wrong in the fills and copies is reported here
    return TRON_OK;
}

// 1 = done, < 0 = an error, 0 = no room: the work space (20 bytes an entry, 32 with host arrays) lies beside the layouts (24 bytes) while they are
// built.  Then nothing is left of the attempt, and the host's way needs the layouts' room only.
static int create_on_device(tron_dataset *ds, const int64_t *h_rowptr, const int32_t *col, const double *val, const double *h_y, int mem, int64_t rows_used)
{
    const int rc = layouts_on_device(ds, h_rowptr, col, val, h_y, mem, rows_used);
    if (rc != TRON_ENOMEM) return rc < 0 ? rc : 1;
    (void)hipGetLastError();
    ds->fwd.release();
    ds->bwd.release();
    return 0;
}

}  // namespace tron

using namespace tron;

// =================================================================== ABI
extern "C" {

const char *tron_last_error(void) { return g_err; }

void tron_dataset_destroy(tron_dataset *ds)
{
    if (!ds) return;
    hipStreamSynchronize(ds->stream);
    dense_device_release(ds);
    csr_resident_release(ds);
    dense_compact_release(ds);
    hipFree(ds->X);
    ds->fwd.release();
    ds->bwd.release();
    hipFree(ds->y); hipFree(ds->y8); hipFree(ds->z); hipFree(ds->zhat); hipFree(ds->Dbuf[0]); hipFree(ds->Dbuf[1]);
    hipFree(ds->partials); hipFree(ds->row_partials); hipFree(ds->unit_scale); hipFree(ds->scal_copy); hipFree(ds->ticket); hipFree(ds->sync_words);
    if (ds->scal_host) hipHostFree(ds->scal_host);
    for (double *p : ds->sv) hipFree(p);
    hipFree(ds->cg_partials);
    ds->prof.destroy();
    delete ds;
}

int tron_dataset_create_csr(int64_t n, int64_t d, const int64_t *rowptr, const int32_t *col, const double *val,
                            const double *y, int mem, void *hip_stream, tron_dataset **out)
{
    if (out) *out = nullptr;
    // the sparse kernels address the gathered vectors through 32-bit byte offsets: n, d < 2^29
    if (!out || !rowptr || !y || n < 1 || d < 1 || n >= (1 << 29) || d >= (1 << 29) ||
        (mem != TRON_MEM_HOST && mem != TRON_MEM_DEVICE)) {
        set_error("tron_dataset_create_csr: bad argument (need 1 <= n,d < 2^29, non-null rowptr/y/out, mem in {0,1})");
        return TRON_EINVAL;
    }
    TRON_TRY(check_device());
    // host arrays are read in place
    std::vector<int64_t> rowptr_copy;
    std::vector<int32_t> col_copy;
    std::vector<double> val_copy, y_copy;
    const int64_t *h_rowptr = rowptr;
    const int32_t *h_col = col;
    const double *h_val = val, *h_y = y;
    if (mem == TRON_MEM_DEVICE) {
        TRON_TRY(fetch(rowptr_copy, rowptr, (size_t)n + 1));
        h_rowptr = rowptr_copy.data();
    }
    if (h_rowptr[0] != 0) { set_error("rowptr[0] = %lld, expected 0", (long long)h_rowptr[0]); return TRON_EINVAL; }
    int64_t rows_used = 0, cols_used = 0;   // rows and columns with entries
    for (int64_t i = 0; i < n; ++i) {
        if (h_rowptr[i + 1] < h_rowptr[i]) { set_error("rowptr decreases at row %lld", (long long)i); return TRON_EINVAL; }
        rows_used += h_rowptr[i + 1] > h_rowptr[i];
    }
    const int64_t nnz = h_rowptr[n];
    if (nnz > 0 && (!col || !val)) { set_error("col/val are null but nnz = %lld", (long long)nnz); return TRON_EINVAL; }
    if (mem == TRON_MEM_DEVICE) {
        TRON_TRY(fetch(y_copy, y, (size_t)n));
        h_y = y_copy.data();
    }
    TRON_TRY(check_labels(h_y, n));
    const bool fwd_partitioned = g_tuning.csr_parts == kColParts ||
                                 (g_tuning.csr_parts == 0 && d * (int64_t)sizeof(double) > (3 << 19) && nnz >= (1 << 22));
    const bool bwd_partitioned = g_tuning.csr_parts == kColParts ||
                                 (g_tuning.csr_parts == 0 && n * (int64_t)sizeof(double) > (3 << 19) && nnz >= (1 << 22));
    const bool on_device = !fwd_partitioned && !bwd_partitioned && nnz > 0 && nnz <= INT32_MAX &&
                           (g_tuning.csr_device_build < 0 ? nnz >= kDeviceBuildNnz : g_tuning.csr_device_build > 0);
    tron_dataset *ds = new (std::nothrow) tron_dataset();
    if (!ds) { set_error("out of host memory"); return TRON_ENOMEM; }
    struct Owner {   // until the handle is the caller's
        tron_dataset *ds;
        ~Owner() { tron_dataset_destroy(ds); }
    } owner{ds};
    ds->n = n; ds->d = d; ds->dense = false; ds->stream = reinterpret_cast<hipStream_t>(hip_stream);
    if (on_device) {
        TRON_TRY(alloc_common(ds));
        const int rc = create_on_device(ds, h_rowptr, col, val, h_y, mem, rows_used);
        TRON_TRY(rc);
        if (rc > 0) TRON_TRY(alloc_row_partials(ds));
        if (rc > 0) {
            *out = ds;
            owner.ds = nullptr;
            return TRON_OK;
        }
    }
    if (mem == TRON_MEM_DEVICE) {
        TRON_TRY(fetch(col_copy, col, (size_t)nnz));
        TRON_TRY(fetch(val_copy, val, (size_t)nnz));
        h_col = col_copy.data();
        h_val = val_copy.data();
    }
    // Columns strictly increasing inside each row and in range; values finite; count per column.  Matrices whose counts fit a
    // cache per thread are walked by several threads, each a block of rows with equal shares of the entries: the blocks' own
    // counts say where each of them places its entries in the transposed copy, instances in ascending order.
    std::vector<int64_t> t_rowptr;
    const unsigned T = (nnz < INT32_MAX && d <= (1 << 19)) ? host_threads(nnz) : 1;
    HostArray<int32_t> block_count;
    std::vector<int64_t> block_row(T + 1, n);
    try {
        t_rowptr.assign((size_t)d + 1, 0);
        if (T > 1) block_count = HostArray<int32_t>((size_t)T * (size_t)d);
    } catch (const std::bad_alloc &) { set_error("out of host memory"); return TRON_ENOMEM; }
    block_row[0] = 0;
    for (unsigned t = 1; t < T; ++t) block_row[t] = std::lower_bound(h_rowptr, h_rowptr + n, nnz / T * t) - h_rowptr;
    struct Fault { int64_t row = -1, col = 0; };   // col < 0: a value that is not finite
    std::vector<Fault> fault(T);
    on_threads(T, [&](unsigned t, unsigned) {
        int32_t *cnt = T > 1 ? block_count.data() + (size_t)t * (size_t)d : nullptr;
        if (cnt) std::fill(cnt, cnt + d, 0);
        for (int64_t i = block_row[t]; i < block_row[t + 1]; ++i) {
            int64_t prev = -1;
            for (int64_t k = h_rowptr[i]; k < h_rowptr[i + 1]; ++k) {
                const int64_t c = h_col[k];
                if (c <= prev || c >= d) { fault[t].row = i; fault[t].col = c; return; }
                if (!std::isfinite(h_val[k])) { fault[t].row = i; fault[t].col = INT64_MIN; return; }
                prev = c;
                if (cnt) cnt[c] += 1;
                else t_rowptr[c + 1] += 1;
            }
        }
    });
    for (const Fault &f : fault) {   // the first in row order
        if (f.row < 0) continue;
        if (f.col == INT64_MIN) set_error("row %lld: non-finite value", (long long)f.row);
        else set_error("row %lld: column index %lld out of order or out of range [0,%lld)", (long long)f.row, (long long)f.col, (long long)d);
        return TRON_EINVAL;
    }
    if (T > 1)
        parallel_ranges(d, (int64_t)T * d, [&](int64_t c0, int64_t c1) {
            for (unsigned t = 0; t < T; ++t)
                for (int64_t c = c0; c < c1; ++c) t_rowptr[c + 1] += block_count[(size_t)t * (size_t)d + c];
        });
    // Unit plans: when both layouts are partitioned and every instance's entries share one value r_i (binary features,
    // optionally scaled per instance, e.g. normalised to unit length), X = diag(r) B with B binary: the layouts keep no
    // values, the row sums of X are multiplied by r afterwards and X^T gathers from r .* (its vector).
    bool unit = g_tuning.csr_unit != 0 && fwd_partitioned && bwd_partitioned;
    std::vector<double> row_value;
    if (unit) {
        try {
            row_value.assign((size_t)n, 1.0);
        } catch (const std::bad_alloc &) { set_error("out of host memory"); return TRON_ENOMEM; }
        for (int64_t i = 0; i < n && unit; ++i) {
            const int64_t k0 = h_rowptr[i], k1 = h_rowptr[i + 1];
            if (k1 > k0) row_value[i] = h_val[k0];
            for (int64_t k = k0 + 1; k < k1; ++k)
                if (h_val[k] != h_val[k0]) { unit = false; break; }
        }
    }
    // Hot-row tiles for the transposed product of large matrices: the features with the most entries (rank r by
    // count -> slice r % 8, slot r / 8) leave the transposed CSR copy and are stored as tiles instead, or without values in windows.
    std::vector<int32_t> slot_code;
    int nhot = 0;
    const bool partitioned = bwd_partitioned;
    if (g_tuning.csr_tiles && partitioned) {
        std::vector<std::pair<int64_t, int32_t>> cand;
        // Without values the entries go to windows (HotWindows), where a feature costs a piece of eight places or more in nearly each of them:
        // those with two entries a window or more.  us of the kernels of the transposed product of 2M x 3M, 123M entries, 128 windows, features from
        // one / two / three / four entries a window on: windows 75 / 62 / 57 / 57, their sums 20 / 15 / 13 / 12, the other features 78 / 90 / 99 / 107.
        const int64_t nwin = unit ? hot_windows_count(n) : 0;
        const int64_t least = unit ? std::max<int64_t>(kTileMinCount, 2 * nwin) : kTileMinCount;
        for (int64_t j = 0; j < d; ++j)
            if (t_rowptr[j + 1] >= least) cand.emplace_back(-t_rowptr[j + 1], (int32_t)j);
        size_t keep = std::min<size_t>(cand.size(), unit ? std::min<int64_t>(kMaxPieceSlots, (1 << 30) / nwin) : (size_t)kTileSlices * kTileSlots);
        std::partial_sort(cand.begin(), cand.begin() + keep, cand.end());
        // A tile spans at most kTileWindow instances, so a slice has about n / kTileWindow of them however few entries
        // they hold, and a tile costs the kernel about as much as 400 entries cost the range kernels: where there are
        // many tiles they must be at least a quarter full on average, or the features stay in the CSR copy.
        if (!unit) {
            int64_t entries = 0;
            for (size_t r = 0; r < keep; ++r) entries -= cand[r].first;
            const int64_t windows = (n + kTileWindow - 1) / kTileWindow * kTileSlices;
            if (windows > 4096 && entries < windows * (kChunk / 4)) keep = 0;
        }
        if (keep > 0) {
            slot_code.assign((size_t)d, -1);
            for (size_t r = 0; r < keep; ++r) {
                slot_code[cand[r].second] = unit ? (int32_t)r : (int32_t)((r % kTileSlices) * kTileSlots + r / kTileSlices);
                t_rowptr[cand[r].second + 1] = 0;   // no entries of this feature in the CSR copy
            }
            nhot = (int)keep;
        }
    }
    // explicit transposed copy (d x n): counting sort by column keeps rows ascending inside each column
    cols_used = nhot;
    for (int64_t j = 0; j < d; ++j) {
        cols_used += t_rowptr[j + 1] > 0;
        t_rowptr[j + 1] += t_rowptr[j];
    }
    const int64_t t_nnz = t_rowptr[d];
    // Both arrays of the copy lie in one block, with room that is never touched.  The C library gives memory back to the system
    // when more than twice its largest block so far is free at the heap's end; with two arrays of 8 and 4 bytes an entry, creation
    // frees more than that, and the next one has every page of its work space mapped again (1.05M entries: 5700 page faults,
    // 6.7 ms a training instead of 5.0; whether it came to that hung on which small object lay behind the arrays).  Blocks above
    // 32 MB are mapped and given back one by one in any case.
    constexpr size_t kEntryBytes = sizeof(double) + sizeof(int32_t), kRoomBytes = 20, kMostBytes = (size_t)30 << 20;
    HostArray<unsigned char> t_block;
    HostArray<int32_t> t_col_alone;
    int32_t *t_col = nullptr;
    double *t_val = nullptr;
    HostArray<int32_t> place;
    std::vector<int64_t> cursor;
    try {
        if (T > 1) place = HostArray<int32_t>((size_t)d);   // here, where running out of memory is an error code, not in the threads
        const size_t entries = (size_t)t_nnz, both = entries * kEntryBytes;
        if (unit || both > kMostBytes) {
            t_col_alone = HostArray<int32_t>(entries);
            if (!unit) t_block = HostArray<unsigned char>(entries * sizeof(double));
            t_col = t_col_alone.data();
        } else {
            t_block = HostArray<unsigned char>(std::min(entries * kRoomBytes, kMostBytes));
            t_col = reinterpret_cast<int32_t *>(t_block.data() + entries * sizeof(double));
        }
        t_val = reinterpret_cast<double *>(t_block.data());
        if (T == 1) cursor.assign(t_rowptr.begin(), t_rowptr.end() - 1);
    } catch (const std::bad_alloc &) { set_error("out of host memory building the transposed copy"); return TRON_ENOMEM; }
    if (T > 1) {
        parallel_ranges(d, (int64_t)T * d, [&](int64_t c0, int64_t c1) {   // the blocks' counts become their first places
            for (int64_t c = c0; c < c1; ++c) place[c] = (int32_t)t_rowptr[c];
            for (unsigned t = 0; t < T; ++t)
                for (int64_t c = c0; c < c1; ++c) {
                    int32_t &cnt = block_count[(size_t)t * (size_t)d + c];
                    const int32_t first = place[c];
                    place[c] += cnt;
                    cnt = first;
                }
        });
        on_threads(T, [&](unsigned t, unsigned) {
            int32_t *at = block_count.data() + (size_t)t * (size_t)d;
            for (int64_t i = block_row[t]; i < block_row[t + 1]; ++i)
                for (int64_t k = h_rowptr[i]; k < h_rowptr[i + 1]; ++k) {
                    const int64_t c = h_col[k];
                    if (nhot && slot_code[c] >= 0) continue;
                    const int64_t pos = at[c]++;
                    t_col[pos] = (int32_t)i;
                    if (!unit) t_val[pos] = h_val[k];
                }
        });
    } else {
        // One host thread per range of features (equal shares of the copy's entries): every thread walks the whole matrix
        // and places the entries of its own features, so the instances stay in ascending order inside a feature and no
        // two threads touch the same cursor.
        const unsigned F = host_threads(t_nnz);
        std::vector<int64_t> bound(F + 1, d);
        bound[0] = 0;
        for (unsigned t = 1; t < F; ++t)
            bound[t] = std::lower_bound(t_rowptr.begin(), t_rowptr.end(), t_nnz / F * t) - t_rowptr.begin();
        for (unsigned t = 1; t <= F; ++t) bound[t] = std::min<int64_t>(d, std::max(bound[t], bound[t - 1]));
        bound[F] = d;
        on_threads(F, [&](unsigned t, unsigned) {
            const int64_t c0 = bound[t], c1 = bound[t + 1];
            if (c0 >= c1) return;
            for (int64_t i = 0; i < n; ++i)
                for (int64_t k = h_rowptr[i]; k < h_rowptr[i + 1]; ++k) {
                    const int64_t c = h_col[k];
                    if (c < c0) continue;
                    if (c >= c1) break;   // columns ascend inside a row
                    if (nhot && slot_code[c] >= 0) continue;
                    const int64_t pos = cursor[c]++;
                    t_col[pos] = (int32_t)i;
                    if (!unit) t_val[pos] = h_val[k];
                }
        });
    }

    int rc = on_device ? TRON_OK : alloc_common(ds);
    if (rc >= 0) {
        // the two layouts are independent of each other: the first is built beside the second where a thread can be had
        int rc_fwd = TRON_OK;
        std::string err_fwd;
        auto build_fwd = [&] {
            hipError_t e = hipSetDevice(ds->device);   // a new thread starts on device 0
            rc_fwd = e != hipSuccess ? hip_fail(e, "hipSetDevice", __FILE__, __LINE__)
                                     : plan_build(ds->fwd, n, d, h_rowptr, h_col, unit ? nullptr : h_val, fwd_partitioned ? kColParts : 1,
                                                  g_tuning.csr_hot != 0, unit, cols_used, ds->stream);
            if (rc_fwd < 0) err_fwd = tron_last_error();
        };
        std::thread beside;
        bool threaded = false;
        try {
            if (nnz >= (1 << 17)) { beside = std::thread(build_fwd); threaded = true; }
        } catch (const std::exception &) {
        }
        if (!threaded) build_fwd();
        rc = plan_build(ds->bwd, d, n, t_rowptr.data(), t_col, unit ? nullptr : t_val, partitioned ? kColParts : 1, false, unit, rows_used,
                        ds->stream);
        if (threaded) beside.join();
        if (rc_fwd < 0) {
            rc = rc_fwd;
            set_error("%s", err_fwd.c_str());
        }
    }
    if (rc >= 0 && nhot) {
        try {
            rc = unit ? hot_windows_build(ds->bwd, h_rowptr, h_col, slot_code, nhot, ds->stream)
                      : hot_tiles_build(ds->bwd, h_rowptr, h_col, h_val, slot_code, nhot, ds->stream);
        } catch (const std::bad_alloc &) { set_error("out of host memory building the hot rows"); rc = TRON_ENOMEM; }
    }
    if (rc >= 0 && unit) {
        hipError_t e = hipMalloc(reinterpret_cast<void **>(&ds->unit_scale), sizeof(double) * (size_t)n);
        if (e == hipSuccess) e = hipMemcpyAsync(ds->unit_scale, row_value.data(), sizeof(double) * (size_t)n, hipMemcpyHostToDevice, ds->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ds->stream);
        if (e != hipSuccess) rc = hip_fail(e, "copy the instances' values", __FILE__, __LINE__);
        ds->fwd.row_scale = ds->unit_scale;
        ds->bwd.col_scale = ds->unit_scale;
    }
    if (rc >= 0) rc = alloc_row_partials(ds);
    if (rc >= 0) {
        hipError_t e = hipMemcpyAsync(ds->y, h_y, sizeof(double) * n, hipMemcpyHostToDevice, ds->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ds->stream);
        if (e != hipSuccess) rc = hip_fail(e, "copy y", __FILE__, __LINE__);
    }
    if (rc < 0) return rc;
    *out = ds;
    owner.ds = nullptr;
    return TRON_OK;
}

int tron_dataset_create_dense_empty(int64_t n, int64_t d, void *hip_stream, tron_dataset **out)
{
    if (out) *out = nullptr;
    if (!out || n < 1 || d < 1 || n > 0x7ffffff0) {
        set_error("tron_dataset_create_dense_empty: bad argument (need 1 <= n < 2^31, d >= 1, non-null out)");
        return TRON_EINVAL;
    }
    if (!dense_supported(d)) { set_error("dense d = %lld not supported (1 <= d <= 512)", (long long)d); return TRON_EINVAL; }
    TRON_TRY(check_device());
    tron_dataset *ds = new (std::nothrow) tron_dataset();
    if (!ds) { set_error("out of host memory"); return TRON_ENOMEM; }
    ds->n = n; ds->d = d; ds->dense = true; ds->stream = reinterpret_cast<hipStream_t>(hip_stream);
    int rc = alloc_common(ds);
    if (rc >= 0) {
        hipError_t e = hipMalloc(reinterpret_cast<void **>(&ds->X), sizeof(double) * (size_t)n * (size_t)d);
        if (e != hipSuccess) rc = hip_fail(e, "allocate X", __FILE__, __LINE__);
    }
    if (rc < 0) { tron_dataset_destroy(ds); return rc; }
    *out = ds;
    return TRON_OK;
}

int tron_dataset_write_rows(tron_dataset *ds, int64_t row0, int64_t nrows, const double *X_chunk, const double *y_chunk, int mem)
{
    if (!ds || !ds->dense || !X_chunk || !y_chunk || row0 < 0 || nrows < 0 || row0 + nrows > ds->n ||
        (mem != TRON_MEM_HOST && mem != TRON_MEM_DEVICE)) {
        set_error("tron_dataset_write_rows: bad argument");
        return TRON_EINVAL;
    }
    if (nrows == 0) return TRON_OK;
    if (mem == TRON_MEM_HOST) {
        TRON_TRY(check_labels(y_chunk, nrows));
        for (int64_t k = 0; k < nrows * ds->d; ++k)
            if (!std::isfinite(X_chunk[k])) { set_error("X has a non-finite entry in row %lld", (long long)(row0 + k / ds->d)); return TRON_EINVAL; }
    } else {
        // the same checks on the device, before anything is copied
        int what = 0;
        TRON_TRY(dense_validate_device(ds, nrows, X_chunk, y_chunk, &what));
        if (what == 1) { set_error("a label in rows [%lld, %lld) is not +1 or -1", (long long)row0, (long long)(row0 + nrows)); return TRON_EINVAL; }
        if (what == 2) { set_error("X has a non-finite entry in rows [%lld, %lld)", (long long)row0, (long long)(row0 + nrows)); return TRON_EINVAL; }
    }
    const hipMemcpyKind kind = (mem == TRON_MEM_HOST) ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    TRON_HIP(hipMemcpyAsync(ds->X + row0 * ds->d, X_chunk, sizeof(double) * (size_t)nrows * (size_t)ds->d, kind, ds->stream));
    std::vector<int8_t> y8;
    if (mem == TRON_MEM_HOST) {
        y8.resize((size_t)nrows);
        for (int64_t i = 0; i < nrows; ++i) y8[i] = (y_chunk[i] > 0.0) ? 1 : -1;
        TRON_HIP(hipMemcpyAsync(ds->y8 + row0, y8.data(), (size_t)nrows, hipMemcpyHostToDevice, ds->stream));
    } else {
        TRON_TRY(dense_labels_from_device(ds, row0, nrows, y_chunk));
    }
    TRON_HIP(hipStreamSynchronize(ds->stream));  // the caller may reuse its buffers on return
    ds->have_D = false;
    return TRON_OK;
}

int tron_dataset_create_dense(int64_t n, int64_t d, const double *X_rowmajor, const double *y, int mem, void *hip_stream,
                              tron_dataset **out)
{
    if (out) *out = nullptr;
    if (!out || !X_rowmajor || !y) { set_error("tron_dataset_create_dense: null argument"); return TRON_EINVAL; }
    tron_dataset *ds = nullptr;
    TRON_TRY(tron_dataset_create_dense_empty(n, d, hip_stream, &ds));
    int rc = tron_dataset_write_rows(ds, 0, n, X_rowmajor, y, mem);
    if (rc < 0) { tron_dataset_destroy(ds); return rc; }
    *out = ds;
    return TRON_OK;
}

int tron_dataset_shape(const tron_dataset *ds, int64_t *n, int64_t *d, int64_t *nnz, int *is_dense)
{
    if (!ds) { set_error("tron_dataset_shape: null handle"); return TRON_EINVAL; }
    if (n) *n = ds->n;
    if (d) *d = ds->d;
    if (nnz) *nnz = ds->dense ? ds->n * ds->d : ds->fwd.nnz;
    if (is_dense) *is_dense = ds->dense ? 1 : 0;
    return TRON_OK;
}

int tron_dataset_stat(const tron_dataset *ds, const char *name, int64_t *value)
{
    if (!ds || !name || !value) { set_error("tron_dataset_stat: null argument"); return TRON_EINVAL; }
    // bytes per launch in the stored format (see PlanBytes); the Hessian-vector call adds the vectors of the call itself
    PlanBytes fb{0, 0, 0, 0, 0, 0}, bb{0, 0, 0, 0, 0, 0};
    int64_t hv_bytes = 0, fun_grad_bytes = 0;
    if (ds->dense) {
        hv_bytes = dense_hv_bytes(ds);
        fun_grad_bytes = dense_fun_grad_bytes(ds);
    } else {
        fb = plan_bytes(ds->fwd);
        bb = plan_bytes(ds->bwd);
        hv_bytes = fb.gather + fb.head + fb.ranges + fb.combine + 8 * ds->n /* D */ +
                   bb.tiles + bb.tile_reduce + bb.ranges + bb.combine + 8 * ds->d /* v as addend */;
        fun_grad_bytes = hv_bytes + 8 * ds->n /* y */ + 8 * ds->n /* zhat and D both written */;
    }
    struct { const char *k; int64_t v; } tab[] = {
        {"fwd_bytes_gather", fb.gather}, {"fwd_bytes_head", fb.head}, {"fwd_bytes_ranges", fb.ranges}, {"fwd_bytes_combine", fb.combine},
        {"bwd_bytes_tiles", bb.tiles}, {"bwd_bytes_tile_reduce", bb.tile_reduce}, {"bwd_bytes_ranges", bb.ranges},
        {"bwd_bytes_combine", bb.combine}, {"hv_bytes", hv_bytes}, {"fun_grad_bytes", fun_grad_bytes},
        {"fwd_parts", ds->dense ? 0 : ds->fwd.P},
        {"bwd_parts", ds->dense ? 0 : ds->bwd.P},
        {"fwd_segmented", (ds->dense || ds->fwd.plain) ? 0 : 1},
        {"bwd_segmented", (ds->dense || ds->bwd.plain) ? 0 : 1},
        {"fwd_single_launch", (!ds->dense && single_sums(ds->fwd)) ? 1 : 0},
        {"bwd_single_launch", (!ds->dense && single_sums(ds->bwd)) ? 1 : 0},
        {"fwd_csr_nnz", ds->dense ? 0 : ds->fwd.nnz},
        {"fwd_head_nnz", (ds->dense || ds->fwd.head < 0) ? 0 : ds->fwd.part_nnz[ds->fwd.head]},
        {"bwd_csr_nnz", ds->dense ? 0 : ds->bwd.nnz},
        {"bwd_tile_nnz", ds->dense ? 0 : ds->bwd.hot.nnz},
        {"bwd_tile_rows", ds->dense ? 0 : ds->bwd.hot.nhot},
        {"bwd_tiles", ds->dense ? 0 : ds->bwd.hot.ntiles_total},
        {"fwd_lds_columns", ds->dense ? 0 : [&] { int64_t t = 0; for (int x = 0; x < kMaxParts; ++x) t += ds->fwd.part_nhot[x]; return t; }()},
        {"dense_grid", ds->dense ? dense_work_units(ds->n, ds->d) : 0},
        {"dense_compact_rows", (ds->dense && ds->have_D && ds->hat_slot == ds->Dcur) ? ds->hat_rows : 0},
        {"unit_values", (!ds->dense && ds->fwd.unit) ? 1 : 0},
        {"solves_in_one_launch", ds->resident.done},
        {"solves_given_up", ds->resident.given_up},
    };
    for (auto &e : tab)
        if (strcmp(e.k, name) == 0) { *value = e.v; return TRON_OK; }
    set_error("tron_dataset_stat: unknown name '%s'", name);
    return TRON_EINVAL;
}

int tron_fun_grad(tron_dataset *ds, int loss, double C, const double *w_dev, double *f_host, double *g_dev)
{
    if (!ds || !w_dev || !f_host || (loss != TRON_LOSS_LR && loss != TRON_LOSS_L2SVM) || !(C > 0.0) || !std::isfinite(C)) {
        set_error("tron_fun_grad: bad argument (null handle/w/f, unknown loss, or C <= 0)");
        return TRON_EINVAL;
    }
    const int slot = ds->have_D ? 1 - ds->Dcur : ds->Dcur;
    if (ds->dense) {
        TRON_TRY(dense_fun_grad(ds, loss, C, w_dev, slot, g_dev));
        TRON_TRY(wait_results(ds));
        ds->active_frac[slot] = ds->scal_host[3] / (double)ds->n;
        ds->active_count[slot] = (int64_t)ds->scal_host[3];
        *f_host = 0.5 * ds->scal_host[1] + C * ds->scal_host[0];
        // stand-alone calls: the compacted copy of the active rows only when the knob forces it
        if (g_tuning.dense_compact > 0 && dense_compact_wanted(ds, slot, 0)) TRON_TRY(dense_compact_build(ds, slot));
    } else {
        TRON_TRY(fun_enqueue(ds, loss, w_dev, slot, true));
        if (g_dev) TRON_TRY(grad_enqueue(ds, C, w_dev, g_dev, 2));
        TRON_TRY(wait_results(ds));
        *f_host = 0.5 * ds->scal_host[1] + C * ds->scal_host[0];
    }
    ds->Dcur = slot;
    ds->have_D = true;
    return TRON_OK;
}

int tron_hv(tron_dataset *ds, double C, const double *v_dev, double *Hv_dev, double *vHv_host)
{
    if (!ds || !v_dev || !Hv_dev || v_dev == Hv_dev || !(C > 0.0) || !std::isfinite(C)) {
        set_error("tron_hv: bad argument (null handle/v/Hv, v aliases Hv, or C <= 0)");
        return TRON_EINVAL;
    }
    if (!ds->have_D) { set_error("tron_hv: no cached D; call tron_fun_grad first"); return TRON_ESTATE; }
    TRON_TRY(hv_enqueue(ds, C, v_dev, Hv_dev));
    if (vHv_host) {
        TRON_TRY(wait_results(ds));
        *vHv_host = ds->scal_host[0];
    }
    return TRON_OK;
}

int tron_profile_enable(tron_dataset *ds, int on)
{
    if (!ds) { set_error("tron_profile_enable: null handle"); return TRON_EINVAL; }
    TRON_HIP(hipStreamSynchronize(ds->stream));
    TRON_TRY(ds->prof.drain());
    ds->prof.on = on != 0;
    for (int s = 0; s < SLOT_COUNT; ++s) { ds->prof.ms[s] = 0; ds->prof.calls[s] = 0; }
    return TRON_OK;
}

int tron_profile_read(tron_dataset *ds, int cap, const char **names, double *ms, int64_t *calls, int *count)
{
    if (!ds || cap < 0) { set_error("tron_profile_read: bad argument"); return TRON_EINVAL; }
    TRON_HIP(hipStreamSynchronize(ds->stream));
    TRON_TRY(ds->prof.drain());
    for (int s = 0; s < SLOT_COUNT && s < cap; ++s) {
        if (names) names[s] = kSlotNames[s];
        if (ms) ms[s] = ds->prof.ms[s];
        if (calls) calls[s] = ds->prof.calls[s];
    }
    if (count) *count = SLOT_COUNT;
    for (int s = 0; s < SLOT_COUNT; ++s) { ds->prof.ms[s] = 0; ds->prof.calls[s] = 0; }
    return TRON_OK;
}

int tron_probe_read_bandwidth(const double *src_dev, int64_t count, int reps, void *hip_stream, double *ms_per_launch,
                              double *checksum)
{
    TRON_TRY(check_device());
    return probe_read(src_dev, count, reps, reinterpret_cast<hipStream_t>(hip_stream), ms_per_launch, checksum);
}

int tron_tuning_set(const char *name, int64_t value)
{
    if (name && strcmp(name, "csr_parts") == 0 && (value == 0 || value == 1 || value == kColParts)) {
        g_tuning.csr_parts = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_hot") == 0 && (value == 0 || value == 1)) {
        g_tuning.csr_hot = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_hot_blocks_per_part") == 0 && value >= 1 && value <= 4096) {
        g_tuning.csr_hot_blocks_per_part = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_range_slots") == 0 && value >= 2 && value <= kHotSlots) {
        g_tuning.csr_range_slots = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_range_blocks_per_part") == 0 && value >= 1 && value <= 1024) {
        g_tuning.csr_range_blocks_per_part = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_head") == 0 && (value == 0 || value == 1)) {
        g_tuning.csr_head = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_tiles") == 0 && (value == 0 || value == 1)) {
        g_tuning.csr_tiles = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_tile_blocks_per_slice") == 0 && value >= 0 && value <= 1024) {
        g_tuning.csr_tile_blocks_per_slice = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_blocks_per_part") == 0 && value >= 1 && value <= 4096) {
        g_tuning.csr_blocks_per_part = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_sell") == 0 && (value == 0 || value == 1)) {
        g_tuning.csr_sell = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_sell_blocks") == 0 && value >= 1 && value <= 4096) {
        g_tuning.csr_sell_blocks = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_segmented") == 0 && value >= -1 && value <= 1) {
        g_tuning.csr_segmented = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_device_build") == 0 && value >= -1 && value <= 1) {
        g_tuning.csr_device_build = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "csr_unit") == 0 && (value == 0 || value == 1)) {
        g_tuning.csr_unit = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "cg_speculate") == 0 && value >= -1 && value <= 1) {
        g_tuning.cg_speculate = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "fuse_reductions") == 0 && value >= -1 && value <= 1) {
        g_tuning.fuse_reductions = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "dense_compact") == 0 && value >= -1 && value <= 1) {
        g_tuning.dense_compact = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "dense_device_driver") == 0 && value >= -1 && value <= 1) {
        g_tuning.dense_device_driver = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "solve_resident") == 0 && value >= -1 && value <= 1) {
        g_tuning.solve_resident = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "solve_wait_us") == 0 && value >= -1 && value <= 10'000'000) {
        g_tuning.solve_wait_us = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "batch_grid") == 0 && value >= 0 && value <= 4096) {
        g_tuning.batch_grid = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "batch_mfma_rows") == 0 && (value == 0 || value == 32 || value == 64)) {
        g_tuning.batch_mfma_rows = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "batch_lean") == 0 && value >= 0 && value <= 1) {
        g_tuning.batch_lean = value;
        return TRON_OK;
    }
    if (name && strcmp(name, "batch_mfma") == 0 && value >= -1 && value <= 1) {
        g_tuning.batch_mfma = value;
        return TRON_OK;
    }
    set_error("tron_tuning_set: unknown knob or value out of range");
    return TRON_EINVAL;
}

int tron_probe_copy_bandwidth(double *dst_dev, const double *src_dev, int64_t count, int reps, void *hip_stream,
                              double *ms_per_launch)
{
    TRON_TRY(check_device());
    return probe_copy(dst_dev, src_dev, count, reps, reinterpret_cast<hipStream_t>(hip_stream), ms_per_launch);
}

}  // extern "C"
