// Sparse layouts of unpartitioned matrices, built on the device: validation of the entries, the transposed copy (a stable sort of the
// entries by column) and the entries' places in a plan.  What is decided per row (chunks, segments, rows longer than a chunk) stays on
// the host, which reads the row offsets only.
//
// Creating a handle from host arrays was the largest part of a training that runs once: 1.05M entries took 4.2 ms on eight host threads (passes over
// the entries with random access, starting the threads, copies of some hundred kilobytes at 2 to 3 GB/s), of which 0.4 ms are the
// transfer of the arrays.  This way: 1.5 ms (2.2 with arrays that the program has not passed before).
#include <algorithm>
#include <cstring>
#include <new>

#include "csr_chunk.h"

namespace tron {

// ------------------------------------------------------------------ pinned memory for small copies
// A copy of pageable memory below some megabytes runs at 2 to 3 GB/s (160 KB 70 us, 1 MB 370 us; 4.2 MB 140 us), one of pinned memory at 25 to
// 50 and without waiting.
void *HostStage::take(size_t bytes)
{
    bytes = (bytes + 255) / 256 * 256;
    if (used_ + bytes > size_) {
        Block *b = new (std::nothrow) Block();
        if (!b) return nullptr;
        const size_t size = std::max<size_t>(bytes, 1 << 20);
        if (hipHostMalloc(&b->p, size, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            delete b;
            return nullptr;
        }
        b->next = blocks_;
        blocks_ = b;
        used_ = 0;
        size_ = size;
    }
    void *p = static_cast<char *>(blocks_->p) + used_;
    used_ += bytes;
    return p;
}

int HostStage::copy(void *dst, const void *src, size_t bytes, hipStream_t st, bool stays)
{
    constexpr size_t kDirect = 4 << 20;   // from here on pageable memory runs at 30 GB/s, and is read for as long as the copy takes
    void *p = bytes >= kDirect ? nullptr : take(bytes);
    if (p) std::memcpy(p, src, bytes);
    TRON_HIP(hipMemcpyAsync(dst, p ? p : src, bytes, hipMemcpyHostToDevice, st));
    if (!p && !stays) TRON_HIP(hipStreamSynchronize(st));
    return TRON_OK;
}

HostStage::~HostStage()
{
    if (blocks_) (void)hipStreamSynchronize(st_);   // the copies have been made
    while (blocks_) {
        Block *b = blocks_;
        blocks_ = b->next;
        (void)hipHostFree(b->p);
        delete b;
    }
}

// ------------------------------------------------------------------ which row an entry belongs to
// first index in 0 .. n with a[index] >= x
template <typename T>
__device__ __forceinline__ int64_t lower_bound(const T *__restrict__ a, int64_t n, T x)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// rows[i] = the last row r < n with start[r] <= at + i, for the kChunk positions from `at` on, those behind the last row's (the padding of a
// chunk) included.  start[n] is the end.  The workgroup's rows are walked, each with positions of its own writing to its first one; where
// there are many more than positions, nearly all of them empty, every position is looked up instead: a run of empty rows may be as long as
// the matrix.
// (us of a creation from 100,000 entries: in 1M rows, the entries in the first 2000, walked 5570, now 2570; 20,000 x 4M, the entries in 4000 columns,
// 24,200 and 5900; on the host 3400 and 10,600.)
__device__ __forceinline__ void rows_of_positions(const int64_t *__restrict__ start, int64_t n, int64_t at, int *rows, int *scan)
{
    const int tid = threadIdx.x;
    const int r0 = (int)lower_bound(start, n, at + 1) - 1, hi = (int)lower_bound(start, n, at + kChunk);
    if (hi - r0 > 8 * kChunk) {
        for (int k = tid; k < kChunk; k += kBlock) rows[k] = (int)lower_bound(start, n, at + k + 1) - 1;
        __syncthreads();
        return;
    }
    for (int k = tid; k < kChunk; k += kBlock) rows[k] = k == 0 ? r0 : -1;
    __syncthreads();
    for (int r = r0 + 1 + tid; r < hi; r += kBlock) {
        const int64_t first = start[r];
        if (start[r + 1] > first) rows[(int)(first - at)] = r;
    }
    __syncthreads();
    // running maximum: eight positions a thread, then over the threads
    int m[8], most = -1;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        most = max(most, rows[8 * tid + e]);
        m[e] = most;
    }
    scan[tid] = most;
    __syncthreads();
#pragma unroll
    for (int step = 1; step < kBlock; step *= 2) {
        const int other = tid >= step ? scan[tid - step] : -1;
        __syncthreads();
        scan[tid] = max(scan[tid], other);
        __syncthreads();
    }
    const int before = tid > 0 ? scan[tid - 1] : -1;
#pragma unroll
    for (int e = 0; e < 8; ++e) rows[8 * tid + e] = max(before, m[e]);
    __syncthreads();
}

// the first entry that is not as it has to be: columns strictly ascending in a row and in range, values finite
__global__ __launch_bounds__(kBlock) void k_expand_rows(int64_t n, int64_t d, int64_t nnz, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                                        const double *__restrict__ val, int32_t *__restrict__ row_of, unsigned long long *__restrict__ bad)
{
    __shared__ int rows[kChunk], scan[kBlock];
    const int64_t at = (int64_t)blockIdx.x * kChunk;
    rows_of_positions(rowptr, n, at, rows, scan);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int i = e * kBlock + threadIdx.x;
        const int64_t k = at + i;
        if (k >= nnz) continue;
        const int r = rows[i], c = col[k];
        const bool first = i > 0 ? rows[i - 1] != r : rowptr[r] == at;
        const int before = first ? -1 : col[k - 1];
        const double v = val[k];
        if (c <= before || c >= d || !(fabs(v) <= 1.7976931348623157e308)) atomicMin(bad, (unsigned long long)k);
        row_of[k] = r;
    }
}

// ------------------------------------------------------------------ stable sort by column, eight bits a pass
// A wavefront has kSortPer consecutive entries; count[digit * waves + wave] of them have the digit.
constexpr int kSortPer = 1024;
constexpr int kDigits = 256;
static_assert(kDigits == kBlock, "a thread per digit");

__global__ __launch_bounds__(kBlock) void k_sort_count(int64_t nnz, int waves, int shift, const int32_t *__restrict__ key, int *__restrict__ count)
{
    __shared__ int mine[kWavesPerBlock][kDigits];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    for (int w = 0; w < kWavesPerBlock; ++w) mine[w][threadIdx.x] = 0;
    __syncthreads();
    const int64_t at = ((int64_t)blockIdx.x * kWavesPerBlock + wv) * kSortPer + lane;
#pragma unroll
    for (int s = 0; s < kSortPer / kWave; ++s) {
        const int64_t k = at + s * kWave;
        if (k < nnz) atomicAdd(&mine[wv][((uint32_t)key[k] >> shift) & (kDigits - 1)], 1);
    }
    __syncthreads();
    for (int w = 0; w < kWavesPerBlock; ++w) {
        const int wave = blockIdx.x * kWavesPerBlock + w;
        if (wave < waves) count[(int64_t)threadIdx.x * waves + wave] = mine[w][threadIdx.x];
    }
}

// counts of a digit (one workgroup each) become the number of its entries in earlier wavefronts; total[digit] = all of them
__global__ __launch_bounds__(kBlock) void k_sort_scan(int waves, int *__restrict__ count, int *__restrict__ total)
{
    __shared__ int part[kWavesPerBlock];
    int *c = count + (int64_t)blockIdx.x * waves;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    int before = 0;
    for (int base = 0; base < waves; base += kBlock) {
        const int i = base + threadIdx.x, v = i < waves ? c[i] : 0;
        const int incl = wave_scan_add(v);
        if (lane == kWave - 1) part[wv] = incl;
        __syncthreads();
        int off = before;
        for (int w = 0; w < wv; ++w) off += part[w];
        if (i < waves) c[i] = off + incl - v;
        for (int w = 0; w < kWavesPerBlock; ++w) before += part[w];
        __syncthreads();
    }
    if (threadIdx.x == 0) total[blockIdx.x] = before;
}

// from == null: the entries' own numbers
__global__ __launch_bounds__(kBlock) void k_sort_scatter(int64_t nnz, int waves, int shift, const int32_t *__restrict__ key, const int32_t *__restrict__ from,
                                                         const int *__restrict__ count, const int *__restrict__ total, int32_t *__restrict__ key_out,
                                                         int32_t *__restrict__ from_out)
{
    __shared__ int place[kWavesPerBlock][kDigits];
    __shared__ int part[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    {   // where the entries of digit threadIdx.x begin
        const int v = total[threadIdx.x], incl = wave_scan_add(v);
        if (lane == kWave - 1) part[wv] = incl;
        __syncthreads();
        int off = incl - v;
        for (int w = 0; w < wv; ++w) off += part[w];
        for (int w = 0; w < kWavesPerBlock; ++w) {
            const int wave = blockIdx.x * kWavesPerBlock + w;
            place[w][threadIdx.x] = off + (wave < waves ? count[(int64_t)threadIdx.x * waves + wave] : 0);
        }
        __syncthreads();
    }
    const int64_t at = ((int64_t)blockIdx.x * kWavesPerBlock + wv) * kSortPer + lane;
    volatile int *mine = place[wv];   // a wavefront's own: its LDS operations complete in order
#pragma unroll 4
    for (int s = 0; s < kSortPer / kWave; ++s) {
        const int64_t k = at + s * kWave;
        const bool valid = k < nnz;
        const int32_t c = valid ? key[k] : 0, f = valid ? (from ? from[k] : (int32_t)k) : 0;
        const int digit = (int)(((uint32_t)c >> shift) & (kDigits - 1));
        uint64_t same = __ballot(valid);   // lanes with the same digit
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (digit >> b) & 1;
            const uint64_t set = __ballot(bit);
            same &= bit ? set : ~set;
        }
        const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)same, 0u));
        const int base = valid ? mine[digit] : 0;
        __builtin_amdgcn_wave_barrier();
        if (valid && rank == 0) mine[digit] = base + __popcll(same);
        __builtin_amdgcn_wave_barrier();
        if (valid) {
            key_out[base + rank] = c;
            from_out[base + rank] = f;
        }
    }
}

// start[c] = the number of entries in columns before c
__global__ __launch_bounds__(kBlock) void k_column_starts(int64_t d, int64_t nnz, const int32_t *__restrict__ key, int64_t *__restrict__ start)
{
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c <= d) start[c] = c < d ? lower_bound(key, nnz, (int32_t)c) : nnz;
}

// ------------------------------------------------------------------ entries to their places
// place[r] = position of row r's first entry, place[rows] = positions in all.  Plain: the places behind a row's entries are filled with zeros at the last
// column before; segments: in the order of load_stream, zeros at column 0.
template <bool SEG>
__global__ __launch_bounds__(kBlock) void k_fill_plan(CsrFill F, int64_t rows_total, int64_t stored, const int64_t *__restrict__ place, int32_t *__restrict__ col,
                                                      double *__restrict__ val)
{
    __shared__ int rows[kChunk], scan[kBlock];
    const int64_t at = (int64_t)blockIdx.x * kChunk;
    rows_of_positions(place, rows_total, at, rows, scan);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int i = e * kBlock + threadIdx.x;
        const int64_t q = at + i;
        if (q >= stored) continue;
        const int r = rows[i];
        const int64_t first = F.start[r], end = F.start[r + 1], j = q - place[r];
        const bool entry = first + j < end;
        int32_t c = 0;
        double v = 0.0;
        if (entry || (!SEG && end > 0)) {
            const int64_t k = entry ? first + j : end - 1;
            const int64_t p = F.from ? F.from[k] : k;
            c = F.index[p];
            if (entry) v = F.val[p];
        }
        if constexpr (SEG) {
            const int64_t chunk = q - i;
            col[chunk + (i >> 2 & 1) * (kChunk / 2) + (i >> 3) * 4 + (i & 3)] = c;
            val[chunk + (i >> 1 & 3) * (kChunk / 4) + (i >> 3) * 2 + (i & 1)] = v;
        } else {
            col[q] = c;
            val[q] = v;
        }
    }
}

int csr_fill_plan(const CsrFill &F, bool segments, int64_t rows, int64_t stored, const int64_t *place_dev, int32_t *col, double *val, hipStream_t st)
{
    const unsigned grid = (unsigned)((stored + kChunk - 1) / kChunk);
    if (grid == 0) return TRON_OK;
    if (segments) hipLaunchKernelGGL(k_fill_plan<true>, dim3(grid), dim3(kBlock), 0, st, F, rows, stored, place_dev, col, val);
    else hipLaunchKernelGGL(k_fill_plan<false>, dim3(grid), dim3(kBlock), 0, st, F, rows, stored, place_dev, col, val);
    TRON_HIP(hipGetLastError());
    return TRON_OK;
}

// ------------------------------------------------------------------ host
void CsrDeviceBuild::release()
{
    hipFree(block);
    if (sorted) hipEventDestroy(sorted);
    block = nullptr;
    sorted = nullptr;
}

// Enqueues the copies, the check and the sort; wait() has the column offsets in t_rowptr, and where the first entry is that is not as it has to be.
int CsrDeviceBuild::begin(int64_t n_, int64_t d_, int64_t nnz_, const int64_t *h_rowptr, const int32_t *col_in, const double *val_in, int mem, HostStage &stage, hipStream_t st)
{
    n = n_;
    d = d_;
    nnz = nnz_;
    const int waves = (int)((nnz + kSortPer - 1) / kSortPer);
    const bool host = mem == TRON_MEM_HOST;
    size_t at = 0;
    auto room = [&](size_t bytes) { const size_t p = at; at += (bytes + 255) / 256 * 256; return p; };
    const size_t o_rowptr = room(8 * (size_t)(n + 1)), o_start = room(8 * (size_t)(d + 1)), o_bad = room(8), o_total = room(4 * kDigits);
    const size_t o_place = room(8 * (size_t)(std::max(n, d) + 1));
    const size_t o_count = room(4 * (size_t)kDigits * waves), o_row = room(4 * (size_t)nnz);
    const size_t o_key[2] = {room(4 * (size_t)nnz), room(4 * (size_t)nnz)}, o_from[2] = {room(4 * (size_t)nnz), room(4 * (size_t)nnz)};
    const size_t o_col = host ? room(4 * (size_t)nnz) : 0, o_val = host ? room(8 * (size_t)nnz) : 0;
    TRON_HIP(hipMalloc(&block, at));
    TRON_HIP(hipEventCreateWithFlags(&sorted, hipEventDisableTiming));
    char *base = static_cast<char *>(block);
    rowptr = reinterpret_cast<int64_t *>(base + o_rowptr);
    start = reinterpret_cast<int64_t *>(base + o_start);
    place = reinterpret_cast<int64_t *>(base + o_place);
    row_of = reinterpret_cast<int32_t *>(base + o_row);
    unsigned long long *bad_dev = reinterpret_cast<unsigned long long *>(base + o_bad);
    int *total = reinterpret_cast<int *>(base + o_total), *count = reinterpret_cast<int *>(base + o_count);
    col = host ? reinterpret_cast<int32_t *>(base + o_col) : col_in;
    val = host ? reinterpret_cast<double *>(base + o_val) : val_in;
    t_rowptr = static_cast<int64_t *>(stage.take(8 * (size_t)(d + 1)));
    bad = static_cast<unsigned long long *>(stage.take(8));
    if (!t_rowptr || !bad) { set_error("out of pinned memory"); return TRON_ENOMEM; }
    const unsigned long long none = ~0ull;
    TRON_TRY(stage.copy(rowptr, h_rowptr, 8 * (size_t)(n + 1), st));
    TRON_TRY(stage.copy(bad_dev, &none, 8, st));
    if (host) {
        TRON_TRY(stage.copy(const_cast<int32_t *>(col), col_in, 4 * (size_t)nnz, st, true));
        TRON_TRY(stage.copy(const_cast<double *>(val), val_in, 8 * (size_t)nnz, st, true));
    }
    hipLaunchKernelGGL(k_expand_rows, dim3((unsigned)((nnz + kChunk - 1) / kChunk)), dim3(kBlock), 0, st, n, d, nnz, rowptr, col, val, row_of, bad_dev);
    TRON_HIP(hipGetLastError());
    const dim3 grid((unsigned)((waves + kWavesPerBlock - 1) / kWavesPerBlock));
    const int32_t *key = col;
    from = nullptr;
    for (int shift = 0, side = 0; shift == 0 || (d - 1) >> shift; shift += 8, side ^= 1) {
        int32_t *key_out = reinterpret_cast<int32_t *>(base + o_key[side]), *from_out = reinterpret_cast<int32_t *>(base + o_from[side]);
        hipLaunchKernelGGL(k_sort_count, grid, dim3(kBlock), 0, st, nnz, waves, shift, key, count);
        hipLaunchKernelGGL(k_sort_scan, dim3(kDigits), dim3(kBlock), 0, st, waves, count, total);
        hipLaunchKernelGGL(k_sort_scatter, grid, dim3(kBlock), 0, st, nnz, waves, shift, key, from, count, total, key_out, from_out);
        TRON_HIP(hipGetLastError());
        key = key_out;
        from = from_out;
    }
    hipLaunchKernelGGL(k_column_starts, dim3((unsigned)(d / kBlock + 1)), dim3(kBlock), 0, st, d, nnz, key, start);
    TRON_HIP(hipGetLastError());
    TRON_HIP(hipMemcpyAsync(t_rowptr, start, 8 * (size_t)(d + 1), hipMemcpyDeviceToHost, st));
    TRON_HIP(hipMemcpyAsync(bad, bad_dev, 8, hipMemcpyDeviceToHost, st));
    TRON_HIP(hipEventRecord(sorted, st));
    return TRON_OK;
}

int CsrDeviceBuild::wait()
{
    TRON_HIP(hipEventSynchronize(sorted));
    return TRON_OK;
}

}  // namespace tron
