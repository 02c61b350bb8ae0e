// Sparse matrix-vector products for both orientations (X and the explicit X^T copy):
//   z = X w,  a1 = D .* (X v)               (Table 1 / Appendix D of the paper: a0 = X v, a1 = D a0)
//   g = w + C X^T zhat,  Hv = v + C X^T a1   (a2 = C X^T a1)
//
// Work is split by nonzeros, not by rows, because row lengths are heavily skewed (Zipf-distributed
// features give the transposed copy rows of length ~n next to millions of length 0/1): a workgroup
// streams one chunk of kChunk nonzeros with 16-byte non-temporal loads that cover whole cache lines,
// multiplies them by the gathered vector entries; the sums of the row
// pieces ("segments") of the chunk come out of a segmented scan (see runs_from_regs).  Rows and segments that fit
// into a chunk are stored so that they never cross a chunk boundary; one longer than a chunk receives the rest
// from the `carry` of the following chunks in a small fix-up kernel, in a fixed order -- nothing is ever added in
// an order that depends on timing, so results are bit-reproducible (the one atomic instruction in use, the LDS
// add of the tile kernel, has a fixed order too).
//
// The gathers decide the speed.  A gather that misses the vector L1 costs an L2 request of its own, and
// a CU keeps only ~100 of them in flight; one that misses L2 as well pulls a 64-byte sector for 8 useful
// bytes.  Large matrices are therefore regrouped by where the gathered element can be kept:
//   - forward orientation: a head partition (the most frequent columns of the whole matrix, served from
//     one LDS table, 16-bit slots, whole rows) and 8 column ranges, workgroup b on range b % 8 so that
//     each XCD's L2 gathers from its own slice of the vector; each range has an LDS table of its own;
//   - transposed orientation: hot-row tiles (see HotTiles: LDS accumulators, gathers from a copy of the tile's
//     columns in LDS), or without values windows of the vector in LDS (see HotWindows), and 8 column ranges for the rest.
// Partitions write one partial sum per segment; combine kernels add a row's partial sums in a fixed
// order and apply the epilogue (loss terms, D scaling, v + C * sum) and the first stage of the scalar
// reductions.
#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <thread>

#include "csr_chunk.h"
#include "host_util.h"

namespace tron {

constexpr int64_t kGatherBytesForPartitioning = 3 << 19;  // 1.5 MiB: larger gather vectors get partitioned
constexpr int64_t kMinNnzForPartitioning = 1 << 22;
constexpr int kHotMinCount = 8;   // columns with fewer entries are not worth an LDS slot

void HotWindows::release()
{
    hipFree(window_of); hipFree(wave_off); hipFree(data); hipFree(row_end); hipFree(pos); hipFree(psums);
    *this = HotWindows();
}

void HotTiles::release()
{
    win.release();
    hipFree(val); hipFree(iloc); hipFree(flags); hipFree(hdr); hipFree(seg_slot); hipFree(slot_of_row);
    hipFree(wg_acc); hipFree(sums);
    *this = HotTiles();
}

void SellHead::release()
{
    hipFree(wave_off); hipFree(data); hipFree(sums); hipFree(pos);
    *this = SellHead();
}

void CsrPlan::release()
{
    hot.release();
    sell.release();
    hipFree(rowptr); hipFree(col); hipFree(col16); hipFree(val); hipFree(row_lo); hipFree(carry);
    hipFree(xs); hipFree(hot_ids); hipFree(hot_x); hipFree(group_base); hipFree(chunk_tab); hipFree(flags); hipFree(row_mask);
    hipFree(row_seg); hipFree(chunk_long); hipFree(long_row); hipFree(long_first); hipFree(long_ticket);
    hipFree(fix_row); hipFree(fix_b0); hipFree(fix_cnt);
    *this = CsrPlan();
}

// stage: the array has been read when the call returns
template <typename T>
static int upload_array(T **dst, const T *src, size_t count, hipStream_t st, HostStage *stage)
{
    *dst = nullptr;
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(dst), sizeof(T) * std::max<size_t>(count, 1)));
    if (!count) return TRON_OK;
    if (stage) return stage->copy(*dst, src, sizeof(T) * count, st);
    TRON_HIP(hipMemcpyAsync(*dst, src, sizeof(T) * count, hipMemcpyHostToDevice, st));
    return TRON_OK;
}
template <typename T>
static int upload(T **dst, const T *src, size_t count, hipStream_t st) { return upload_array(dst, src, count, st, nullptr); }

// row_lo / fix-up lists of the plain layout.  rp[r] = position of row r's first entry, rp[rows] = entries stored.
static void plan_chunks(const int64_t *rp, int64_t rows, int nchunks, std::vector<int32_t> &row_lo, std::vector<int32_t> &fix_row,
                        std::vector<int32_t> &fix_b0, std::vector<int32_t> &fix_cnt)
{
    // row_lo[c] = first row r with rp[r] >= c*kChunk; row_lo[nchunks] = rows
    row_lo.resize((size_t)nchunks + 1);
    int64_t r = 0;
    for (int c = 0; c < nchunks; ++c) {
        const int64_t start = (int64_t)c * kChunk;
        while (r < rows && rp[r] < start) ++r;
        row_lo[c] = (int32_t)r;
    }
    row_lo[0] = 0;
    row_lo[nchunks] = (int32_t)rows;
    // chunk c >= 1 begins inside row row_lo[c]-1 iff rp[row_lo[c]] > c*kChunk  (rp[rows] = entries stored)
    for (int c = 1; c < nchunks; ++c) {
        const int64_t start = (int64_t)c * kChunk;
        const int32_t lo = row_lo[c];
        if (lo >= 1 && rp[lo] > start) {
            const int32_t row = lo - 1;
            if (!fix_row.empty() && fix_row.back() == row) {
                fix_cnt.back() += 1;
            } else {
                fix_row.push_back(row);
                fix_b0.push_back(c);
                fix_cnt.push_back(1);
            }
        }
    }
}

// Where entry e of a chunk is stored.  Thread t of a kernel owns entries 8t .. 8t+7 of a chunk, and its loads cover whole
// cache lines: the columns come as two pieces of four (16 bytes), the values as four pieces of two, piece m of all threads
// together.  The 16-bit slots of a head partition or a tile are 16 bytes per thread and stay in order.
static inline int64_t col_pos(int64_t q) { const uint32_t e = (uint32_t)q & (kChunk - 1); return q - e + ((e >> 2 & 1) * (kChunk / 2) + (e >> 3) * 4 + (e & 3)); }
static inline int64_t val_pos(int64_t q) { const uint32_t e = (uint32_t)q & (kChunk - 1); return q - e + ((e >> 1 & 3) * (kChunk / 4) + (e >> 3) * 2 + (e & 1)); }

int csr_plan_build(CsrPlan &A, int64_t rows, int64_t cols, const int64_t *h_rowptr, const int32_t *h_col,
                   const double *h_val, int parts, bool hot, bool unit, int64_t cols_used, hipStream_t st, const CsrFill *fill, HostStage *stage)
{
    auto upload = [&](auto **dst, const auto *src, size_t count, hipStream_t s) { return upload_array(dst, src, count, s, stage); };
    // the arrays on the host may go
    auto arrays_done = [&]() -> int {
        if (!stage) TRON_HIP(hipStreamSynchronize(st));
        return TRON_OK;
    };
    A.rows = rows;
    A.cols = cols;
    A.nnz = h_rowptr[rows];
    A.unit = unit;
    if (parts <= 0)
        parts = (cols * (int64_t)sizeof(double) > kGatherBytesForPartitioning && A.nnz >= kMinNnzForPartitioning) ? kColParts : 1;
    if (parts > kColParts) parts = kColParts;
    A.P = parts;
    A.plain = (parts == 1);
    std::vector<int32_t> row_lo, fix_row, fix_b0, fix_cnt;

    if (A.unit && A.P == 1) { set_error("internal: unit plan without partitions"); return TRON_EINVAL; }
    if (A.plain && g_tuning.csr_segmented != 0) {
        // The plain kernel gives a chunk's rows groups of g = 256 / (rows starting in the chunk) lanes, one thread per row
        // when there are more than 128: a row of hundreds of entries among many short ones (the middle of a Zipf
        // distribution, in the transposed copy) then keeps one thread adding for tens of microseconds.  Count, per chunk,
        // the additions the busiest thread would make; beyond 96 the segment layout (scans, no per-row loops) is used.
        bool segmented = g_tuning.csr_segmented > 0;
        int64_t r = 0;
        const int64_t nchunks = (A.nnz + kChunk - 1) / kChunk;
        for (int64_t c = 0; c < nchunks && !segmented; ++c) {
            const int64_t start = c * kChunk, end = std::min<int64_t>(A.nnz, start + kChunk);
            while (r < rows && h_rowptr[r] < start) ++r;
            int64_t nrows = 0, longest = 0;
            for (int64_t q = r; q < rows && h_rowptr[q] < end; ++q) {
                ++nrows;
                longest = std::max<int64_t>(longest, std::min<int64_t>(h_rowptr[q + 1], end) - h_rowptr[q]);
            }
            int64_t g = 1;
            while (g < kWave && nrows * (g * 2) <= kBlock) g *= 2;
            if ((longest + g - 1) / g > 96) segmented = true;
        }
        if (segmented) A.plain = false;
    }
    hot = hot && A.P > 1;   // LDS tables belong to the column ranges of large matrices
    if (A.plain) {
        // A row that fits into a chunk never straddles a chunk boundary: one that would is moved to the start of the next
        // chunk.  The gap it leaves is counted to the row before, filled with zeros at that row's last column (they add
        // 0 times an entry of the vector the row reads anyway).  Only rows longer than a chunk are still completed by the
        // fix-up kernel; for matrices of short rows that launch disappears.
        std::vector<int64_t> rp((size_t)rows + 1);
        int64_t at = 0;
        for (int64_t r = 0; r < rows; ++r) {
            const int64_t len = h_rowptr[r + 1] - h_rowptr[r];
            if (len > 0 && len <= kChunk && at % kChunk + len > kChunk) at = (at / kChunk + 1) * kChunk;
            rp[r] = at;
            at += len;
        }
        rp[rows] = at;
        const int64_t stored = at;
        const HostArray<int32_t> pcol(fill ? 0 : (size_t)stored);
        const HostArray<double> pval(fill ? 0 : (size_t)stored);
        if (!fill) parallel_ranges(rows, stored, [&](int64_t r0, int64_t r1) {
            for (int64_t r = r0; r < r1; ++r) {
                const int64_t k0 = h_rowptr[r], k1 = h_rowptr[r + 1];
                int64_t q = rp[r];
                for (int64_t k = k0; k < k1; ++k, ++q) { pcol[q] = h_col[k]; pval[q] = h_val[k]; }
                if (q == rp[r + 1]) continue;
                const int32_t last_col = k1 > 0 ? h_col[k1 - 1] : 0;   // of the last row with entries up to here
                for (; q < rp[r + 1]; ++q) { pcol[q] = last_col; pval[q] = 0.0; }
            }
        });
        const int64_t nb64 = std::max<int64_t>(1, (stored + kChunk - 1) / kChunk);
        if (nb64 > 0x7ffffff0) { set_error("matrix too large: %lld chunks", (long long)nb64); return TRON_EINVAL; }
        A.nblocks = (int)nb64;
        A.part_base[0] = 0; A.part_nnz[0] = stored; A.part_chunk0[0] = 0; A.part_nchunks[0] = A.nblocks;
        A.max_chunks = A.nblocks;
        plan_chunks(rp.data(), rows, A.nblocks, row_lo, fix_row, fix_b0, fix_cnt);
        for (int c = 0; c < A.nblocks; ++c) A.max_rows = std::max(A.max_rows, row_lo[c + 1] - row_lo[c]);
        TRON_TRY(upload(&A.rowptr, rp.data(), (size_t)rows + 1, st));
        if (fill) {
            TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.col), sizeof(int32_t) * (size_t)std::max<int64_t>(stored, 1)));
            TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.val), sizeof(double) * (size_t)std::max<int64_t>(stored, 1)));
            TRON_TRY(csr_fill_plan(*fill, false, rows, stored, A.rowptr, A.col, A.val, st));
        } else {
            TRON_TRY(upload(&A.col, pcol.data(), (size_t)stored, st));
            TRON_TRY(upload(&A.val, pval.data(), (size_t)stored, st));
        }
        TRON_TRY(arrays_done());
    } else {
        const int P = A.P;
        std::vector<int64_t> colcount((size_t)cols + 1, 0);
        if (P > 1)   // a single range needs no counts
            for (int64_t k = 0; k < A.nnz; ++k) colcount[h_col[k] + 1]++;
        // Head partition: the kHotSlots most frequent columns of the whole matrix, when they hold a good part of
        // the nonzeros.  Their entries need no locality in L2 (one LDS table serves them all), so they are not
        // split by column range: one segment per row instead of one per row and range.
        std::vector<uint8_t> part_of((size_t)cols, 0);
        std::vector<int32_t> slot_of, hot_ids;
        std::vector<std::pair<int64_t, int32_t>> cand;
        int64_t head_nnz = 0;
        // unit plans keep the head partition as sorted slices (SellHead) instead of chunks, with a larger table
        const bool want_sell = A.unit && g_tuning.csr_sell != 0;
        A.head_slots = want_sell ? kSellSlots : kHotSlots;
        if (hot) {
            A.range_slots = (int)std::min<int64_t>(kHotSlots, std::max<int64_t>(2, g_tuning.csr_range_slots / 2 * 2));
            slot_of.assign((size_t)cols, -1);
            hot_ids.assign((size_t)P * kHotSlots + A.head_slots, 0);
        }
        if (hot && g_tuning.csr_head) {
            for (int64_t j = 0; j < cols; ++j)
                if (colcount[j + 1] >= kHotMinCount) cand.emplace_back(-colcount[j + 1], (int32_t)j);
            const size_t keep = std::min<size_t>(cand.size(), (size_t)A.head_slots);
            std::partial_sort(cand.begin(), cand.begin() + keep, cand.end());
            for (size_t k = 0; k < keep; ++k) head_nnz -= cand[k].first;
            if (head_nnz * 4 >= A.nnz) {
                A.head = P;
                A.part_nhot[P] = (int)keep;
                A.part_nnz[P] = head_nnz;
                for (size_t k = 0; k < keep; ++k) {
                    part_of[cand[k].second] = (uint8_t)P;
                    slot_of[cand[k].second] = (int32_t)k;
                    hot_ids[(size_t)P * kHotSlots + k] = cand[k].second;
                    colcount[cand[k].second + 1] = 0;   // not counted in the ranges below
                }
            }
        }
        const bool sell = want_sell && A.head >= 0;
        const int NP = (A.head >= 0 && !sell) ? P + 1 : P;   // chunked partitions in all
        const int64_t range_nnz = A.nnz - ((A.head >= 0) ? head_nnz : 0);
        // column ranges with equal nonzero counts (head columns excluded): bound[x] = first column of range x
        for (int64_t j = 0; j < cols; ++j) colcount[j + 1] += colcount[j];
        std::vector<int64_t> bound(P + 1, cols);
        bound[0] = 0;
        for (int x = 1; x < P; ++x) {
            const int64_t target = range_nnz / P * x;
            bound[x] = std::lower_bound(colcount.begin(), colcount.end(), target) - colcount.begin();
            if (bound[x] > cols) bound[x] = cols;
            if (bound[x] < bound[x - 1]) bound[x] = bound[x - 1];
        }
        for (int x = 0; x < P; ++x)
            for (int64_t j = bound[x]; j < bound[x + 1]; ++j)
                if (part_of[j] != P || A.head < 0) part_of[j] = (uint8_t)x;
        for (int x = 0; x < P; ++x) A.part_nnz[x] = P > 1 ? colcount[bound[x + 1]] - colcount[bound[x]] : A.nnz;
        for (int x = 0; x < NP; ++x)
            if (A.part_nnz[x] > 0x7ffffff0) { set_error("partition too large for 32-bit offsets"); return TRON_EINVAL; }
        // LDS-resident columns of a range: its kHotSlots most frequent columns with at least kHotMinCount entries
        if (hot) {
            for (int x = 0; x < P; ++x) {
                cand.clear();
                for (int64_t j = bound[x]; j < bound[x + 1]; ++j) {
                    const int64_t cnt = colcount[j + 1] - colcount[j];   // 0 for head columns
                    if (cnt >= kHotMinCount) cand.emplace_back(-cnt, (int32_t)j);
                }
                const size_t keep = std::min<size_t>(cand.size(), (size_t)A.range_slots);
                std::partial_sort(cand.begin(), cand.begin() + keep, cand.end());
                A.part_nhot[x] = (int)keep;
                for (size_t k = 0; k < keep; ++k) {
                    slot_of[cand[k].second] = (int32_t)k;
                    hot_ids[(size_t)x * kHotSlots + k] = cand[k].second;
                }
            }
        }
        if (P == 1) A.cold_cols = cols_used;
        for (int64_t j = 0; j < cols; ++j)   // head columns have count 0 here
            if (colcount[j + 1] > colcount[j] && !(hot && slot_of[j] >= 0)) A.cold_cols++;
        std::vector<int64_t>().swap(colcount);
        // per-(partition,row) entry counts -> offsets; non-empty pairs are the segments.  A segment that would straddle a
        // chunk boundary is moved to the start of the next chunk (the gap it leaves is padding that reaches no sum), so
        // that a chunk never continues a row of the chunk before and no carry / fix-up pass is needed; only a segment
        // longer than a whole chunk is still split.
        std::vector<int32_t> rp32((size_t)NP * (rows + 1), 0);    // start of (x, r) relative to the partition
        std::vector<int32_t> len32((size_t)NP * rows, 0);         // its number of entries
        std::vector<int32_t> head_cnt(sell ? (size_t)rows : 0, 0);   // entries of the row in a head kept as sorted slices
        // one table for the passes over the entries below: partition in the upper half, LDS slot + 1 (0: none) in the lower
        std::vector<int32_t> code_of(P > 1 ? (size_t)cols : 0);
        for (int64_t j = 0; P > 1 && j < cols; ++j) code_of[j] = ((int32_t)part_of[j] << 16) | ((hot && slot_of[j] >= 0) ? slot_of[j] + 1 : 0);
        parallel_ranges(rows, P == 1 ? rows : A.nnz, [&](int64_t r0, int64_t r1) {
            if (P == 1) {
                for (int64_t r = r0; r < r1; ++r) len32[(size_t)r] = (int32_t)(h_rowptr[r + 1] - h_rowptr[r]);
                return;
            }
            for (int64_t r = r0; r < r1; ++r)
                for (int64_t k = h_rowptr[r]; k < h_rowptr[r + 1]; ++k) {
                    const int x = code_of[h_col[k]] >> 16;
                    if (x < NP) len32[(size_t)x * rows + r]++;
                    else if (sell && x == P) head_cnt[r]++;
                }
        });
        // a head kept as sorted slices: the slots of a row's head entries, row after row (filled with the ranges below)
        std::vector<int64_t> head_off(sell ? (size_t)rows + 1 : 0, 0);
        for (int64_t r = 0; sell && r < rows; ++r) head_off[r + 1] = head_off[r] + head_cnt[r];
        std::vector<uint16_t> head_slot(sell ? (size_t)head_off[rows] : 0);
        std::vector<uint16_t> mask((size_t)rows, 0);
        int64_t pos = 0, nseg_total = 0;
        int chunk = 0;
        A.max_chunks = 0;
        for (int x = 0; x < NP; ++x) {
            int32_t *rp = rp32.data() + (size_t)x * (rows + 1);
            const int32_t *ln = len32.data() + (size_t)x * rows;
            int64_t nseg = 0, at = 0;
            for (int64_t r = 0; r < rows; ++r) {
                const int64_t len = ln[r];
                if (len > 0) {
                    mask[r] |= (uint16_t)(1u << x);
                    ++nseg;
                    if (len <= kChunk && at % kChunk + len > kChunk) at = (at / kChunk + 1) * kChunk;
                }
                rp[r] = (int32_t)at;
                at += len;
                if (at > 0x7ffffff0) { set_error("partition too large for 32-bit offsets"); return TRON_EINVAL; }
            }
            rp[rows] = (int32_t)at;
            A.part_base[x] = pos;
            A.part_seg0[x] = nseg_total;
            A.part_chunk0[x] = chunk;
            A.part_nchunks[x] = (int)std::max<int64_t>(1, (at + kChunk - 1) / kChunk);
            if (x < P) A.max_chunks = std::max(A.max_chunks, A.part_nchunks[x]);
            chunk += A.part_nchunks[x];
            pos += (int64_t)A.part_nchunks[x] * kChunk;
            nseg_total += nseg;
        }
        A.nblocks = chunk;
        if (nseg_total > 0x7ffffff0) { set_error("too many row segments for 32-bit indexing"); return TRON_EINVAL; }
        // entries partition-major; inside a row the entries of one range are contiguous and stay ordered
        size_t stored_cols = (size_t)pos;
        HostArray<int32_t> pcol(fill ? 0 : (size_t)pos);
        HostArray<double> pval(A.unit || fill ? 0 : (size_t)pos);
        if (!fill) parallel_ranges(pos, pos, [&](int64_t q0, int64_t q1) {
            std::fill(pcol.data() + q0, pcol.data() + q1, 0);
            if (!A.unit) std::fill(pval.data() + q0, pval.data() + q1, 0.0);
        });
        if (!fill) parallel_ranges(rows, A.nnz, [&](int64_t r0, int64_t r1) {   // a row's places belong to that row alone
            int64_t cursor[kMaxParts + 1];
            if (P == 1) {
                for (int64_t r = r0; r < r1; ++r) {
                    int64_t q = rp32[(size_t)r];
                    for (int64_t k = h_rowptr[r]; k < h_rowptr[r + 1]; ++k, ++q) {
                        pcol[col_pos(q)] = h_col[k];
                        pval[val_pos(q)] = h_val[k];
                    }
                }
                return;
            }
            for (int64_t r = r0; r < r1; ++r) {
                for (int x = 0; x < NP; ++x) cursor[x] = A.part_base[x] + rp32[(size_t)x * (rows + 1) + r];
                int64_t hq = sell ? head_off[r] : 0;
                for (int64_t k = h_rowptr[r]; k < h_rowptr[r + 1]; ++k) {
                    const int32_t code = code_of[h_col[k]];
                    const int x = code >> 16, slot1 = code & 0xffff;
                    if (x >= NP) {   // head entries of a plan with sorted slices
                        if (sell && x == P) head_slot[hq++] = (uint16_t)(slot1 - 1);
                        continue;
                    }
                    const int64_t q = cursor[x]++;
                    pcol[x < P ? col_pos(q) : q] = slot1 ? ~(slot1 - 1) : h_col[k];   // the head's become 16-bit slots below
                    if (!A.unit) pval[val_pos(q)] = h_val[k];
                }
            }
        });
        // segment tables
        std::vector<int32_t> seg_row((size_t)std::max<int64_t>(nseg_total, 1));
        std::vector<int4> tab((size_t)chunk);
        std::vector<uint8_t> flags((size_t)chunk * kBlock, 0);   // per chunk: one bit per entry, set on the last entry of a segment
        for (int x = 0; x < NP; ++x) {
            const int32_t *rp = rp32.data() + (size_t)x * (rows + 1);
            const int32_t *ln = len32.data() + (size_t)x * rows;
            const int nch = A.part_nchunks[x];
            // the segments of this partition, in row order, with start/end positions relative to the partition
            int64_t m = 0;               // segment counter (partition-relative)
            int c = 0;                   // chunk that owns the segments being emitted
            int4 t = make_int4(0, 0, 0, 0);
            auto close_chunk = [&](int next_first_seg, int64_t next_seg_start) {
                tab[A.part_chunk0[x] + c] = t;
                ++c;
                const int64_t cstart = (int64_t)c * kChunk;
                const int64_t off = std::min<int64_t>(std::max<int64_t>(next_seg_start - cstart, 0), kChunk);
                t = make_int4(next_first_seg, 0, (int)off, 0);
            };
            for (int64_t r = 0; r < rows; ++r) {
                const int64_t rs = rp[r], re = rs + ln[r];
                if (re == rs) continue;
                while (rs >= (int64_t)(c + 1) * kChunk) close_chunk((int)m, rs);   // this segment starts in a later chunk
                seg_row[A.part_seg0[x] + m] = (int32_t)r;
                t.y += 1;
                // the row's piece in each chunk it touches ends with a flag; continuation chunks go to the fix-up list
                const int c_last = (int)((re - 1) / kChunk);
                for (int ck = c; ck <= c_last; ++ck) {
                    const int64_t pe = std::min<int64_t>(re, (int64_t)(ck + 1) * kChunk) - 1 - (int64_t)ck * kChunk;
                    flags[((size_t)A.part_chunk0[x] + ck) * kBlock + pe / 8] |= (uint8_t)(1u << (pe % 8));
                }
                if (c_last > c) {
                    fix_row.push_back((int32_t)(A.part_seg0[x] + m));   // partitioned plans: the segment's slot in the partial sums
                    fix_b0.push_back(A.part_chunk0[x] + c + 1);
                    fix_cnt.push_back(c_last - c);
                }
                ++m;
            }
            while (c < nch - 1) close_chunk((int)m, (int64_t)rp[rows]);
            tab[A.part_chunk0[x] + c] = t;
        }
        // first_off of a chunk inside or at the end of a split row: the chunk-relative end of that row
        // (set above from the start of the next segment; for chunks wholly inside one row that start lies
        // beyond the chunk and clips to kChunk, which is right)
        if (hot) {
            TRON_TRY(upload(&A.hot_ids, hot_ids.data(), hot_ids.size(), st));   // unused slots: column 0
            TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.hot_x), sizeof(double) * hot_ids.size()));
        }
        if (sell) {
            // ---- sorted slices of the head partition
            const std::vector<int32_t> &cnt = head_cnt;   // counted with the segment lengths above
            struct Slice { int32_t len8; int64_t first; };   // first: position of its 64 rows in `order`
            std::vector<int32_t> order((size_t)rows);
            std::vector<Slice> slices;
            for (int64_t w0 = 0; w0 < rows; w0 += kSellWindow) {
                const int64_t w1 = std::min<int64_t>(rows, w0 + kSellWindow);
                for (int64_t r = w0; r < w1; ++r) order[r] = (int32_t)r;
                std::stable_sort(order.begin() + w0, order.begin() + w1, [&](int32_t a, int32_t b) { return cnt[a] > cnt[b]; });
                for (int64_t s0 = w0; s0 < w1; s0 += kWave) {
                    const int32_t longest = cnt[order[s0]];
                    if (longest == 0) break;   // the rest of the window has no head entries
                    slices.push_back({(longest + 7) / 8, s0});
                }
            }
            std::stable_sort(slices.begin(), slices.end(), [](const Slice &a, const Slice &b) { return a.len8 > b.len8; });
            SellHead &S = A.sell;
            S.on = true;
            S.nslices = (int)slices.size();
            S.nwaves = (int)std::max<int64_t>(1, std::min<int64_t>(g_tuning.csr_sell_blocks, 4096)) * kWavesPerBlock;
            // longest first, each slice to the wavefront with the least work so far (ties: the lower wavefront)
            std::vector<std::vector<int32_t>> mine((size_t)S.nwaves);
            {
                std::vector<std::pair<int64_t, int32_t>> heap;   // (-load, -wave): the top is the least loaded, lowest wave
                for (int w = 0; w < S.nwaves; ++w) heap.emplace_back(0, -w);
                std::make_heap(heap.begin(), heap.end());
                for (size_t i = 0; i < slices.size(); ++i) {
                    std::pop_heap(heap.begin(), heap.end());
                    auto &top = heap.back();
                    mine[(size_t)(-top.second)].push_back((int32_t)i);
                    top.first -= slices[i].len8;
                    std::push_heap(heap.begin(), heap.end());
                }
            }
            std::vector<int64_t> wave_off((size_t)S.nwaves + 1);
            std::vector<int64_t> goff(slices.size());    // header group of each slice (in stored order)
            std::vector<int32_t> stored(slices.size());  // stored position -> index into slices
            int64_t groups = 0;
            int32_t sl = 0;
            std::vector<int64_t> null_groups;   // padding of every stream to a whole number of kSellAhead groups
            for (int w = 0; w < S.nwaves; ++w) {
                wave_off[w] = groups;
                for (int32_t i : mine[(size_t)w]) {
                    stored[sl] = i;
                    goff[sl] = groups;
                    groups += 1 + slices[i].len8;
                    ++sl;
                }
                while ((groups - wave_off[w]) % kSellAhead) null_groups.push_back(groups++);
            }
            wave_off[S.nwaves] = groups;
            S.ngroups = groups;
            for (int64_t r = 0; r < rows; ++r) S.nrows_with_entries += cnt[r] > 0;
            std::vector<uint16_t> data((size_t)std::max<int64_t>(groups, 1) * kWave * 8, (uint16_t)kSellSlots);
            for (int64_t gpad : null_groups)
                for (int l = 0; l < kWave; ++l) {
                    const int32_t hdr[4] = {-1, 0, 0, 0};   // a header of a slice without groups
                    std::memcpy(&data[((size_t)gpad * kWave + l) * 8], hdr, sizeof(hdr));
                }
            parallel_ranges((int64_t)slices.size(), groups * kWave, [&](int64_t p0, int64_t p1) {   // a slice's groups belong to it alone
            for (int64_t p = p0; p < p1; ++p) {
                const Slice &sc = slices[stored[p]];
                const int64_t w1 = std::min<int64_t>(rows, (sc.first / kSellWindow + 1) * (int64_t)kSellWindow);
                for (int l = 0; l < kWave; ++l) {
                    int32_t hdr[4] = {-1, sc.len8, 0, 0};
                    const int64_t pos = sc.first + l;
                    const int32_t r = (pos < w1) ? order[pos] : -1;
                    if (r >= 0 && cnt[r] > 0) {
                        hdr[0] = (int32_t)pos;   // sums are kept in sorted order
                        // entry j of the row: group 1 + j / 8 of the slice, lane l, place j % 8
                        const uint16_t *hs = head_slot.data() + head_off[r];
                        for (int j = 0; j < cnt[r]; ++j) data[((size_t)(goff[p] + 1 + j / 8) * kWave + l) * 8 + j % 8] = hs[j];
                    }
                    std::memcpy(&data[((size_t)goff[p] * kWave + l) * 8], hdr, sizeof(hdr));
                }
            }
            });
            {
                std::vector<int32_t> pos_of((size_t)rows);
                for (int64_t q = 0; q < rows; ++q) pos_of[order[q]] = (int32_t)q;
                TRON_TRY(upload(&S.pos, pos_of.data(), pos_of.size(), st));
                TRON_HIP(hipStreamSynchronize(st));
            }
            TRON_TRY(upload(&S.wave_off, wave_off.data(), wave_off.size(), st));
            TRON_TRY(upload(&S.data, data.data(), data.size(), st));
            TRON_HIP(hipMalloc(reinterpret_cast<void **>(&S.sums), sizeof(double) * (size_t)rows));
            TRON_HIP(hipMemsetAsync(S.sums, 0, sizeof(double) * (size_t)rows, st));
            TRON_HIP(hipStreamSynchronize(st));
        } else if (A.head >= 0) {
            // the head partition is the last one: its columns go to col16, the ranges' stay in col
            const size_t h0 = (size_t)A.part_base[A.head];
            std::vector<uint16_t> c16((size_t)pos - h0, 0);
            // padding: slot 0 (value 0; in a unit plan the padding lies behind the last flagged entry of the partition, and
            // what follows the last flag of a chunk never reaches a sum)
            for (size_t k = h0; k < (size_t)pos; ++k) c16[k - h0] = (uint16_t)(pcol[k] < 0 ? ~pcol[k] : 0);
            TRON_TRY(upload(&A.col16, c16.data(), c16.size(), st));
            TRON_HIP(hipStreamSynchronize(st));
            stored_cols = h0;
        }
        if (fill) {   // one range
            std::vector<int64_t> place(rp32.begin(), rp32.begin() + rows + 1);
            TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.col), sizeof(int32_t) * (size_t)pos));
            TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.val), sizeof(double) * (size_t)pos));
            TRON_TRY(stage->copy(fill->place, place.data(), sizeof(int64_t) * place.size(), st));
            TRON_TRY(csr_fill_plan(*fill, true, rows, pos, fill->place, A.col, A.val, st));
        } else TRON_TRY(upload(&A.col, pcol.data(), stored_cols, st));
        if (!fill && !A.unit) TRON_TRY(upload(&A.val, pval.data(), (size_t)pos, st));
        if (A.unit) TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.xs), sizeof(double) * (size_t)(cols + 1)));
        A.nseg_total = nseg_total;
        // A single range: the kernel applies the epilogue itself where every chunk has a bounded number of rows (the empty ones
        // among them) and the sums it leaves are few enough to be added up by the kernel after it.
        if (P == 1) {
            const int nlong = (int)fix_row.size();
            std::vector<int32_t> rl((size_t)chunk + 1);
            int64_t r = 0, most = 0;
            for (int c = 0; c < chunk; ++c) {
                while (r < rows && rp32[r] < (int64_t)c * kChunk) ++r;
                rl[c] = c ? (int32_t)r : 0;
                if (c) most = std::max<int64_t>(most, rl[c] - rl[c - 1]);
            }
            rl[chunk] = (int32_t)rows;
            most = std::max<int64_t>(most, rows - rl[chunk - 1]);
            A.max_rows = (int)std::min<int64_t>(most, 0x7fffffff);
            if (most <= 4 * kChunk && chunk + nlong <= kDirectMaxSums) {
                std::vector<int32_t> row_seg((size_t)rows, -1);
                for (int64_t m = 0; m < nseg_total; ++m) row_seg[seg_row[m]] = (int32_t)m;
                std::vector<int2> chunk_long((size_t)chunk, make_int2(-1, -1));
                std::vector<int4> long_row((size_t)nlong);
                for (int l = 0; l < nlong; ++l) {
                    long_row[l] = make_int4(seg_row[fix_row[l]], fix_b0[l], fix_cnt[l], 0);
                    chunk_long[fix_b0[l] - 1].y = l;
                    for (int k = 0; k < fix_cnt[l]; ++k) chunk_long[fix_b0[l] + k].x = l;
                }
                TRON_TRY(upload(&A.row_lo, rl.data(), rl.size(), st));
                TRON_TRY(upload(&A.row_seg, row_seg.data(), row_seg.size(), st));
                TRON_TRY(upload(&A.chunk_long, chunk_long.data(), chunk_long.size(), st));
                if (nlong) {
                    TRON_TRY(upload(&A.long_row, long_row.data(), long_row.size(), st));
                    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.long_first), sizeof(double) * nlong));
                    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.long_ticket), sizeof(unsigned) * nlong));
                    TRON_HIP(hipMemsetAsync(A.long_ticket, 0, sizeof(unsigned) * nlong, st));
                }
                TRON_TRY(arrays_done());
                A.direct = true;
            }
        }
        if (!A.direct) {   // what the combine kernels read
            // group_base[G].first[x] = first segment of partition x whose row is >= 64 G (see sum_parts)
            A.ngroups = (rows + kWave - 1) / kWave;
            std::vector<GroupBase> gbase((size_t)A.ngroups);
            std::memset(gbase.data(), 0, sizeof(GroupBase) * gbase.size());
            for (int x = 0; x < NP; ++x) {
                const int64_t s0 = A.part_seg0[x], s1 = (x + 1 < NP) ? A.part_seg0[x + 1] : nseg_total;
                int64_t m = s0;
                for (int64_t G = 0; G < A.ngroups; ++G) {
                    while (m < s1 && seg_row[m] < G * kWave) ++m;
                    gbase[(size_t)G].first[x] = (int32_t)m;
                }
            }
            TRON_TRY(upload(&A.group_base, gbase.data(), gbase.size(), st));
            TRON_TRY(upload(&A.row_mask, mask.data(), mask.size(), st));
            TRON_TRY(arrays_done());   // gbase goes out of scope
        }
        TRON_TRY(upload(&A.chunk_tab, tab.data(), tab.size(), st));
        TRON_TRY(upload(&A.flags, flags.data(), flags.size(), st));
        TRON_TRY(arrays_done());
    }
    A.nfix = (int)fix_row.size();
    A.fix_max_cnt = 0;
    for (int32_t c : fix_cnt) A.fix_max_cnt = std::max(A.fix_max_cnt, (int)c);
    if (A.plain) TRON_TRY(upload(&A.row_lo, row_lo.data(), row_lo.size(), st));
    if (!A.direct) {   // (its long rows are in long_row)
        TRON_TRY(upload(&A.fix_row, fix_row.data(), fix_row.size(), st));
        TRON_TRY(upload(&A.fix_b0, fix_b0.data(), fix_b0.size(), st));
        TRON_TRY(upload(&A.fix_cnt, fix_cnt.data(), fix_cnt.size(), st));
    }
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&A.carry), sizeof(double) * A.nblocks));
    TRON_HIP(hipMemsetAsync(A.carry, 0, sizeof(double) * A.nblocks, st));
    TRON_TRY(arrays_done());   // the host vectors above go out of scope
    return TRON_OK;
}

// ------------------------------------------------------------------ chunk kernel
// What happens to a row's sum z:
//   PLAIN  out = z;   SCALE  out = aux z;   AXPY  out = aux + alpha z (no aux: 1 + alpha z), and the row's share of out . (self ?
//   out : aux);   LR / SVM  the loss terms at z with aux = the labels: out = zhat, D, and the row's loss.
enum { EPI_PLAIN = 0, EPI_SCALE = 1, EPI_AXPY = 2, EPI_LR = 3, EPI_SVM = 4 };
struct EpiArgs {
    double *out;
    const double *aux;
    double alpha;
    bool self;
    double *D;
    double *red;   // per-workgroup sums of the shares; null: not wanted
    Finish fin;
};

template <int EPI>
__device__ __forceinline__ double row_aux(const EpiArgs &A, int64_t r)
{
    if (EPI == EPI_PLAIN) return 0.0;
    if (EPI == EPI_AXPY) return A.aux ? A.aux[r] : 1.0;
    return A.aux[r];
}

// returns the row's share of the sum
template <int EPI>
__device__ __forceinline__ double finish_row(const EpiArgs &A, int64_t r, double z, double aux)
{
    if constexpr (EPI == EPI_LR || EPI == EPI_SVM) {
        double a, zh, Di;
        loss_terms_dev<EPI == EPI_LR ? TRON_LOSS_LR : TRON_LOSS_L2SVM>(z, aux, a, zh, Di);
        A.out[r] = zh;
        A.D[r] = Di;
        return a;
    } else if constexpr (EPI == EPI_AXPY) {
        const double o = fma(A.alpha, z, aux);
        A.out[r] = o;
        return o * (A.self ? o : aux);
    } else {
        A.out[r] = EPI == EPI_SCALE ? aux * z : z;
        return 0.0;
    }
}

// With HOT, a negative stored column c means "entry ~c of the workgroup's LDS table" (the most frequent
// columns of the partition, copied from x once per workgroup).
template <bool HOT>
__device__ __forceinline__ double gather(const double *__restrict__ x, const double *table, int c)
{
    if (!HOT) return load_elem(x, c);
    // two separate accesses (an LDS read and a lane-masked global load), not one flat load of a selected address
    const double hot = table[(c < 0) ? ~c : 0];
    double cold = 0.0;
    if (c >= 0) cold = load_elem(x, c);
    return (c < 0) ? hot : cold;
}

// Rows lo + base, lo + base + 1, ... below lo + nrows, kPasses passes of one row a thread; returns acc with their epilogue's sums
// added.  Everything the passes need is asked for at once, without a branch between the loads (with one, each pass waits for
// its own, and the 1.05M nonzeros of the rcv1-shaped matrix, whose chunks do not come here, take 10.3 us instead of 8.9).
template <int EPI, int kPasses>
__device__ __forceinline__ double short_rows(const EpiArgs &A, const int64_t *__restrict__ rp, const double *prod, int lo, int nrows, int base,
                                             int64_t start, int64_t end, double acc)
{
    int64_t rs[kPasses], re[kPasses];
    double aux[kPasses];
#pragma unroll
    for (int j = 0; j < kPasses; ++j) {
        const int ri = base + j * kBlock + threadIdx.x;
        const int64_t r = (int64_t)lo + (ri < nrows ? ri : nrows - 1);
        rs[j] = rp[r];
        re[j] = rp[r + 1];
        aux[j] = row_aux<EPI>(A, r);
    }
#pragma unroll
    for (int j = 0; j < kPasses; ++j) {
        const int ri = base + j * kBlock + threadIdx.x;
        if (ri < nrows) {
            const int k0 = (int)(rs[j] - start);
            const int k1 = (int)(((re[j] < end) ? re[j] : end) - start);
            double s = 0.0;
            for (int k = k0; k < k1; ++k) s += prod[k];
            acc += finish_row<EPI>(A, (int64_t)lo + ri, s, aux[j]);
        }
    }
    return acc;
}

// Plain CSR: one workgroup per chunk of nonzeros, the epilogue applied directly.  The chunk's row range, and the offsets and
// the addends of the rows a thread starts with, are asked for before the gathers: asked for where they are used, after the
// products are in LDS, they added three memory latencies to a kernel that is little else (9.6 us for the 1.05M nonzeros of
// the rcv1-shaped matrix).
template <int EPI, bool SQ>
__global__ __launch_bounds__(kBlock) void k_csr_spmv(int64_t nnz, const int64_t *__restrict__ rowptr,
                                                     const int32_t *__restrict__ col, const double *__restrict__ val,
                                                     const int32_t *__restrict__ row_lo, const double *__restrict__ x, EpiArgs A,
                                                     double *__restrict__ carry)
{
    __shared__ __align__(16) double prod[kChunk];
    __shared__ double lds[kWavesPerBlock];
    const int tid = threadIdx.x;
    const int64_t start = (int64_t)blockIdx.x * kChunk;
    const int64_t end = (start + kChunk < nnz) ? start + kChunk : nnz;
    const int64_t *__restrict__ rp = rowptr;
    const int lo = row_lo[blockIdx.x], nrows = row_lo[blockIdx.x + 1] - lo;
    const bool full = end - start == kChunk;
    // thread t takes entries m*512 + 2t, m*512 + 2t + 1: every load instruction covers whole cache lines
    v2i c[4];
    v2d v[4];
    if (full) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int64_t k = start + m * (kChunk / 4) + tid * 2;
            c[m] = __builtin_nontemporal_load(reinterpret_cast<const v2i *>(col + k));
            v[m] = __builtin_nontemporal_load(reinterpret_cast<const v2d *>(val + k));
        }
    }
    // rows that start in this chunk: groups of g lanes per row, g = 256 / (number of rows) rounded
    // down to a power of two (so one pass covers them whenever there are at most 256 rows)
    int g = 1;
    while (g < kWave && nrows * (g * 2) <= kBlock) g *= 2;
    const int sub = tid & (g - 1);
    const int rows_per_pass = kBlock / g;
    const int ri0 = tid / g;
    int64_t rs0 = 0, re0 = 0;
    double aux0 = 0.0;
    if (ri0 < nrows) {
        rs0 = rp[lo + ri0];
        re0 = rp[lo + ri0 + 1];
        aux0 = row_aux<EPI>(A, lo + ri0);
    }
    const int64_t next_start = (blockIdx.x > 0) ? rp[lo] : start;   // rp[rows] == nnz
    if (full) {
        double xg[4][2];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            xg[m][0] = load_elem(x, c[m].x);
            xg[m][1] = load_elem(x, c[m].y);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            double2 p;
            p.x = (SQ ? v[m].x * v[m].x : v[m].x) * xg[m][0];
            p.y = (SQ ? v[m].y * v[m].y : v[m].y) * xg[m][1];
            *reinterpret_cast<double2 *>(prod + m * (kChunk / 4) + tid * 2) = p;
        }
    } else {
        for (int k = tid; k < kChunk; k += kBlock) {
            const int64_t kk = start + k;
            prod[k] = (kk < end) ? (SQ ? val[kk] * val[kk] : val[kk]) * load_elem(x, col[kk]) : 0.0;
        }
    }
    __syncthreads();

    // carry: the part of row lo-1 that lies in this chunk (wavefront 0)
    if (next_start > start && tid < kWave) {
        const int len = (int)(((next_start < end) ? next_start : end) - start);
        double s = 0.0;
        for (int k = tid; k < len; k += kWave) s += prod[k];
        s = wave_sum(s);
        if (tid == 0) carry[blockIdx.x] = s;
    }

    double acc = 0.0;
    if (g == 1 && nrows > kBlock) {
        // Many short rows (the tail of a Zipf-distributed transposed copy: a thousand rows of one or two entries in a
        // chunk): one thread per row, and the row offsets of eight passes are fetched together -- a pass that waited
        // for its own two offsets first cost a memory round trip each, eight or more per chunk.  Four or two where no more
        // are left: chunks of rows with five to eight entries have not many more than 256.  Forward products, always eight passes /
        // this: 1.5M rows of 5 entries 29.5 / 24.7 us, 1M of about 6 26.2 / 22.5, 1.5M of about 8 37.4 / 34.3, of 2 18.2 / 17.2,
        // 800,000 of 3 17.7 / 16.6, 1M of one 15.1 / 15.2.
        int base = 0;
        for (; nrows - base > 4 * kBlock; base += 8 * kBlock) acc = short_rows<EPI, 8>(A, rp, prod, lo, nrows, base, start, end, acc);
        if (nrows - base > 2 * kBlock) acc = short_rows<EPI, 4>(A, rp, prod, lo, nrows, base, start, end, acc);
        else if (base < nrows) acc = short_rows<EPI, 2>(A, rp, prod, lo, nrows, base, start, end, acc);
    } else {
        for (int base = 0; base < nrows; base += rows_per_pass) {
            const int ri = base + ri0;
            if (base > 0 && ri < nrows) {
                rs0 = rp[lo + ri];
                re0 = rp[lo + ri + 1];
                aux0 = row_aux<EPI>(A, lo + ri);
            }
            double s = 0.0;
            if (ri < nrows) {
                const int k0 = (int)(rs0 - start);
                const int k1 = (int)(((re0 < end) ? re0 : end) - start);
                for (int k = k0 + sub; k < k1; k += g) s += prod[k];
            }
            s = group_sum(s, g);
            if (ri < nrows && sub == 0) acc += finish_row<EPI>(A, (int64_t)lo + ri, s, aux0);
        }
    }
    if (A.red) {
        acc = block_sum(acc, lds);
        if (tid == 0) store_shared(A.red + blockIdx.x, acc);
        finish_partials<1>(A.fin, A.red, 0, lds);
    }
}

struct PartArgs {
    int64_t base[kMaxParts];
    int64_t nnz[kMaxParts];
    int64_t seg0[kMaxParts];
    int chunk0[kMaxParts];
    int nchunks[kMaxParts];
    int nhot[kMaxParts];
    int P;
    int slots;   // LDS table entries per workgroup (a multiple of 2; the tables are stored kHotSlots apart)
};

// Partitioned layout, persistent workgroups: workgroup (partition xp, q) walks chunks q, q + Q, ... of its
// partition (Q = gridDim / P).  Everything the next chunk needs -- the col/val stream, the chunk's table entry,
// its segment end offsets and the row ids this thread will write -- is fetched into registers while the current
// chunk is being reduced, so HBM latency is paid once per workgroup, not once per chunk.
// With HOT the partition's most frequent columns are first copied from x into an LDS table; entries of those
// columns are stored as ~slot and never touch the vector cache.
// Stream registers of one chunk: thread t holds its own entries 8t .. 8t+7 (see col_pos / val_pos).  Every load instruction of
// a wavefront covers whole consecutive cache lines: one that reads 16 of every 32 bytes is served in 64-byte requests, twice
// as many, and the number of requests a CU keeps in flight is what bounds it.
template <bool HEAD, bool UNIT>
struct StreamRegs {
    v4i c[HEAD ? 1 : 2];        // HEAD: eight 16-bit LDS slots
    v2d v[UNIT ? 1 : 4];        // UNIT: the entries carry no values (see CsrPlan::unit)
};

template <bool HEAD, bool UNIT>
__device__ __forceinline__ void load_stream(StreamRegs<HEAD, UNIT> &s, const void *__restrict__ col, const double *__restrict__ val, int64_t start)
{
    if constexpr (HEAD) {
        s.c[0] = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(static_cast<const uint16_t *>(col) + start + threadIdx.x * 8));
    } else {
#pragma unroll
        for (int m = 0; m < 2; ++m)
            s.c[m] = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(static_cast<const int32_t *>(col) + start + m * (kChunk / 2) + threadIdx.x * 4));
    }
    if constexpr (!UNIT) {
#pragma unroll
        for (int m = 0; m < 4; ++m) s.v[m] = __builtin_nontemporal_load(reinterpret_cast<const v2d *>(val + start + m * kQuarter + threadIdx.x * 2));
    }
}

// the products of the thread's eight entries
template <bool HOT, bool HEAD, bool SQ, bool UNIT>
__device__ __forceinline__ void products(const StreamRegs<HEAD, UNIT> &r, const double *__restrict__ x, const double *table, double (&p)[8])
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if constexpr (HEAD) {
            const unsigned two = (unsigned)r.c[0][e / 2];
            p[e] = table[e % 2 ? two >> 16 : two & 0xffffu];
        } else {
            p[e] = gather<HOT>(x, table, r.c[e / 4][e % 4]);
        }
    }
    if constexpr (!UNIT) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double v = r.v[e / 2][e % 2];
            p[e] *= SQ ? v * v : v;
        }
    }
}

// flag byte of the calling thread: bit e = entry 8*tid + e is the last of its segment
__device__ __forceinline__ unsigned load_flags(const uint8_t *__restrict__ flags /* of this chunk */)
{
    return flags[threadIdx.x];
}

// Segment sums of the chunk whose products are p (the thread's eight): the sums of the owned segments go to out[0 .. nseg) in
// segment order (one coalesced store per 64 segments; the partial sums of a plan are stored segment by segment, not by row:
// see sum_parts), the piece of a row that started in an earlier chunk to *carry_slot.  Two barriers; the caller
// adds one before it reuses `prod`.
__device__ __forceinline__ void chunk_segments(double *prod, const unsigned flags, const int nseg, const bool continued,
                                               double *__restrict__ out, double *__restrict__ carry_slot, double (&p)[8])
{
    double cin;
    int idx0;
    runs_from_regs(prod, threadIdx.x, flags, p, cin, idx0);
    double *outv = prod + kOutOffset;
    int i = idx0 - (continued ? 1 : 0);
    bool first = true;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if ((flags >> e) & 1u) {
            const double v = first ? p[e] + cin : p[e];
            if (i < 0) *carry_slot = v;
            else outv[i] = v;
            first = false;
            ++i;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSegPasses; ++j) {
        const int sidx = (int)threadIdx.x + kBlock * j;
        if (j * kBlock < nseg && sidx < nseg) out[sidx] = outv[sidx];
    }
}

// A single range of segments whose kernel applies the epilogue itself (see CsrPlan::direct): one workgroup per chunk.  A chunk's
// rows (the empty ones among them) are row_lo[c] .. row_lo[c + 1]; row_seg says which segment a row is, or -1.  A row longer
// than a chunk is added up by the workgroup that finishes last among its chunks, in a fixed order; its share of the sum
// goes to a slot of its own (red[workgroups + row's index among the long ones]), so no sum depends on timing.  The launches
// this saves -- the fix-up of the long rows and the combine kernel -- took 4.0 and 6.2 us of the 22 us of a product with the
// transposed copy of the rcv1-shaped matrix.
struct DirectPtrs {
    const int32_t *col;
    const double *val;
    const int4 *chunk_tab;
    const uint8_t *flags;
    const int32_t *row_lo, *row_seg;
    const int2 *chunk_long;    // per chunk: index of the long row that continues into it / that starts in it, or -1
    const int4 *long_row;      // {row, first chunk it continues into, number of those, unused}
    double *carry;             // per chunk: the piece of the long row that continues into it
    double *long_first;        // per long row: its piece in the chunk it starts in
    unsigned *long_ticket;     // per long row (zero between launches)
};

template <int EPI, bool SQ>
__global__ __launch_bounds__(kBlock) void k_csr_direct(DirectPtrs P, int nlong, const double *__restrict__ x, EpiArgs A)
{
    constexpr int kAhead = 8;   // a chunk of short rows has up to 2048, and empty ones
    __shared__ __align__(16) double prod[kProdDoubles];
    __shared__ double lds[kWavesPerBlock];
    __shared__ double piece;
    const int tid = threadIdx.x, c = blockIdx.x;
    StreamRegs<false, false> s;
    load_stream(s, P.col, P.val, (int64_t)c * kChunk);
    const unsigned flags = P.flags[(int64_t)c * kBlock + tid];
    const int lo = P.row_lo[c], hi = P.row_lo[c + 1];
    const int4 tab = P.chunk_tab[c];
    const int2 lr = P.chunk_long[c];
    int seg[kAhead];
    double aux[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
        const int r = lo + j * kBlock + tid;
        seg[j] = r < hi ? P.row_seg[r] : -1;
        aux[j] = r < hi ? row_aux<EPI>(A, r) : 0.0;
    }
    double p[8], cin;
    products<false, false, SQ, false>(s, x, nullptr, p);
    int idx0;
    runs_from_regs(prod, threadIdx.x, flags, p, cin, idx0);
    double *outv = prod + kOutOffset;
    {
        int i = idx0 - (tab.z > 0 ? 1 : 0);
        bool first = true;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if ((flags >> e) & 1u) {
                const double v = first ? p[e] + cin : p[e];
                if (i < 0) piece = v;
                else outv[i] = v;
                first = false;
                ++i;
            }
        }
    }
    __syncthreads();
    const int starts_long = lr.y >= 0 ? tab.x + tab.y - 1 : -1;   // the segment that is only a long row's first piece
    double acc = 0.0;
    // the last wavefront sees to the long rows while the others start on the chunk's own
    if ((lr.x >= 0 || lr.y >= 0) && tid >= kBlock - kWave) {
        const int lane = tid & (kWave - 1);
        if (lane == 0) {
            if (lr.x >= 0) store_shared(P.carry + c, piece);
            if (lr.y >= 0) store_shared(P.long_first + lr.y, outv[tab.y - 1]);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the pieces have arrived
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int l = q ? lr.y : lr.x;
            if (l < 0) continue;   // uniform
            const int4 R = P.long_row[l];
            unsigned ticket = 0;
            if (lane == 0) ticket = __hip_atomic_fetch_add(P.long_ticket + l, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((int)__builtin_amdgcn_readfirstlane(ticket) != R.z) continue;
            double z = 0.0;
            for (int k = lane; k < R.z; k += kWave) z += load_shared(P.carry + R.y + k);
            z = wave_sum(z) + load_shared(P.long_first + l);
            if (lane == 0) {
                const double share = finish_row<EPI>(A, R.x, z, row_aux<EPI>(A, R.x));
                if (A.red) store_shared(A.red + gridDim.x + l, share);
                P.long_ticket[l] = 0u;
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // before this workgroup's own ticket, if there is one
    }
    for (int base = lo; base < hi; base += kAhead * kBlock) {
        if (base > lo) {
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const int r = base + j * kBlock + tid;
                seg[j] = r < hi ? P.row_seg[r] : -1;
                aux[j] = r < hi ? row_aux<EPI>(A, r) : 0.0;
            }
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const int r = base + j * kBlock + tid;
            if (r < hi && !(starts_long >= 0 && seg[j] == starts_long)) acc += finish_row<EPI>(A, r, seg[j] >= 0 ? outv[seg[j] - tab.x] : 0.0, aux[j]);
        }
    }
    if (A.red) {
        acc = block_sum(acc, lds);
        if (tid == 0) store_shared(A.red + c, acc);
        finish_partials<1>(A.fin, A.red, 0, lds, nlong);
    }
}

// hot_x[k] = x[hot_ids[k]]: the LDS tables of all partitions, so that a workgroup fills its table with 128 line
// requests instead of 4096 gathers
__global__ __launch_bounds__(kBlock) void k_gather_hot(int n, const int32_t *__restrict__ hot_ids, const double *__restrict__ x,
                                                       double *__restrict__ hot_x)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k < n) hot_x[k] = x[hot_ids[k]];
}

// A table entry that every thread of the workgroup needs, fetched with a vector load.  A scalar load would be counted
// by the same counter as the LDS operations, so the wait for LDS before the next barrier would also wait for it --
// a full memory latency in every iteration of the persistent loops, which prefetch these entries two chunks ahead.
__device__ __forceinline__ int4 load_uniform(const int4 *__restrict__ p)
{
    return p[lane_zero()];
}

struct PartPtrs {   // device arrays of one partitioned plan (or of its head partition, pre-offset where noted)
    const void *col;           // int32 columns of the ranges, or the head's 16-bit slots
    const double *val;
    const int4 *chunk_tab;
    const uint8_t *flags;
    const double *hot_x;       // x at the LDS-resident columns, kHotSlots per partition (null without LDS tables)
    double *partial;           // partial sums, one per segment of the plan
    double *carry;
};

// Partitioned layout, persistent workgroups: workgroup (partition xp, q) walks chunks q, q + Q, ... of its
// partition.  Everything the next chunk needs -- the col/val stream, the chunk's table entry, its flags and the row
// ids this thread will write -- is fetched into registers while the current chunk is being reduced, so HBM latency
// is paid once per workgroup, not once per chunk.
// SQ: the values are squared (sum_i x_ij^2 a_i, for the diagonal of the Hessian)
template <bool HOT, bool HEAD, bool SQ, bool UNIT>
__device__ __forceinline__ void part_body(double *prod, double *table, const PartArgs &pa, const int xp, const int q, const int Q,
                                          const int64_t rows, const PartPtrs &pp, const double *__restrict__ x)
{
    const int tid = threadIdx.x;
    const int nchunks = pa.nchunks[xp];
    if (q >= nchunks) return;
    if (HOT) {
        // the vector entries of this partition's LDS-resident columns, gathered once per call by k_gather_hot
        const double2 *__restrict__ src = reinterpret_cast<const double2 *>(pp.hot_x + (size_t)xp * kHotSlots);
        for (int k = tid; k < pa.slots / 2; k += kBlock) reinterpret_cast<double2 *>(table)[k] = src[k];
        __syncthreads();
    }
    // col/val are padded to whole chunks (zeros)
    const void *col = HEAD ? static_cast<const void *>(static_cast<const uint16_t *>(pp.col) + pa.base[xp])
                           : static_cast<const void *>(static_cast<const int32_t *>(pp.col) + pa.base[xp]);
    const double *val = UNIT ? nullptr : pp.val + pa.base[xp];
    const int4 *__restrict__ tabs = pp.chunk_tab + pa.chunk0[xp];
    const uint8_t *__restrict__ flags = pp.flags + (int64_t)pa.chunk0[xp] * kBlock;
    double *partial = pp.partial + pa.seg0[xp];
    double *carry = pp.carry + pa.chunk0[xp];

    int c = q;
    int4 tab = load_uniform(tabs + c);
    int4 tab_n = load_uniform(tabs + ((c + Q < nchunks) ? c + Q : c));
    StreamRegs<HEAD, UNIT> cur;
    load_stream(cur, col, val, (int64_t)c * kChunk);
    unsigned fl = load_flags(flags + (int64_t)c * kBlock);

    for (; c < nchunks; c += Q) {
        double p[8];
        products<HOT, HEAD, SQ, UNIT>(cur, x, table, p);
        // Only now fetch the next chunk (clamped index: always the same loads): nothing below waits for these
        // registers, so they stay in flight during the segment sums and are waited for at the top of the next
        // iteration.
        __builtin_amdgcn_sched_barrier(0);
        const int cn = (c + Q < nchunks) ? c + Q : c;
        const int cnn = (cn + Q < nchunks) ? cn + Q : cn;
        StreamRegs<HEAD, UNIT> nxt;
        load_stream(nxt, col, val, (int64_t)cn * kChunk);
        const unsigned fl_n = load_flags(flags + (int64_t)cn * kBlock);
        const int4 tab_nn = load_uniform(tabs + cnn);
        __builtin_amdgcn_sched_barrier(0);
        chunk_segments(prod, fl, tab.y, tab.z > 0, partial + tab.x, carry + c, p);
        __syncthreads();  // the totals and the parked sums are reused by the next chunk
        cur = nxt;
        fl = fl_n;
        tab = tab_n;
        tab_n = tab_nn;
    }
}

// Head partition of a unit plan stored as sorted slices (see SellHead).  A wavefront reads its own contiguous stream of
// groups (64 lanes x 16 bytes = eight 16-bit slots per lane); lane l sums row l of the current slice and writes the
// sum when the slice ends.  The loads of the next kSellAhead groups are always in flight, also across the ends of
// slices (they are short: the pipeline must not drain there); a slice's row ids and length come in its header group.  No barrier after the table is filled, no segment bookkeeping.  The sum of a row is
// (entries 0, 2, 4, ...) + (entries 1, 3, 5, ...), each in storage order.
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// the stream of one wavefront: groups g0 .. g1 of data, gathers from the table in LDS
__device__ __forceinline__ void sell_stream(const double *table, const int64_t *__restrict__ wave_off, int w, const uint16_t *__restrict__ data,
                                            double *__restrict__ sums)
{
    const int lane = threadIdx.x & (kWave - 1);
    // everything that steers the loop is kept in scalar registers: a branch on a vector condition would make the compiler
    // wait for every load in flight where the paths join
    const int64_t g0 = uniform64(wave_off[w]);
    const int64_t total = uniform64(wave_off[w + 1]) - g0;   // a multiple of kSellAhead
    if (total <= 0) return;
    const v4i *__restrict__ p = reinterpret_cast<const v4i *>(data) + g0 * kWave + lane;
    v4i buf[kSellAhead];
#pragma unroll
    for (int a = 0; a < kSellAhead; ++a) buf[a] = __builtin_nontemporal_load(p + (int64_t)a * kWave);
    int left = 0;    // groups left in the current slice (0: the next group is a header)
    int row = -1;
    double e0 = 0.0, e1 = 0.0;
    // buffer a holds group g + a: the body is unrolled over the buffers, so no buffer is ever copied (a copy would have to
    // wait for the load that fills its source); everything a slice needs arrives through this one stream, in order
    for (int64_t g = 0; g < total; g += kSellAhead) {
#pragma unroll
        for (int a = 0; a < kSellAhead; ++a) {
            const v4i cur = buf[a];
            const int64_t nx = g + a + kSellAhead;
            buf[a] = __builtin_nontemporal_load(p + ((nx < total) ? nx : total - 1) * kWave);
            if (left == 0) {   // a header (a slice without groups is padding)
                row = cur[0];
                left = __builtin_amdgcn_readfirstlane(cur[1]);
            } else {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const unsigned two = (unsigned)cur[m];
                    e0 += table[two & 0xffffu];
                    e1 += table[two >> 16];
                }
                if (--left == 0) {   // the slice ends
                    if (row >= 0) sums[row] = e0 + e1;
                    e0 = 0.0;
                    e1 = 0.0;
                }
            }
        }
    }
}

constexpr int kSellWaves = kSellBlock / kWave;

__global__ __launch_bounds__(kSellBlock) void k_head_sell(int nwaves, const int64_t *__restrict__ wave_off, const uint16_t *__restrict__ data,
                                                         const double *__restrict__ hot_x, double *__restrict__ sums)
{
    __shared__ __align__(16) double table[kSellSlots + 2];
    {
        const double2 *__restrict__ src = reinterpret_cast<const double2 *>(hot_x);
        for (int k = threadIdx.x; k < kSellSlots / 2; k += kSellBlock) reinterpret_cast<double2 *>(table)[k] = src[k];
        if (threadIdx.x == 0) table[kSellSlots] = 0.0;   // the padding slot
        __syncthreads();
    }
    const int w = blockIdx.x * kSellWaves + threadIdx.x / kWave;
    if (w < nwaves) sell_stream(table, wave_off, w, data, sums);
}

// Hot rows of a unit plan (see HotWindows): the table is the window of x.  Bound by LDS gathers like the head's kernel: 62 us for 106M entries
// of 23,000 features over 2M instances in 128 windows.  The tiles that hold such rows in plans with values (k_hot_tiles: segmented scans,
// accumulators in LDS) took 105 us without values, for 103M entries of 16,384 features.
__global__ __launch_bounds__(kSellBlock) void k_window_sell(const int32_t *__restrict__ window_of, int width, int64_t cols, const int64_t *__restrict__ wave_off,
                                                           const uint16_t *__restrict__ data, const double *__restrict__ x, double *__restrict__ psums)
{
    __shared__ __align__(16) double table[kSellSlots + 2];
    const int64_t c0 = (int64_t)window_of[blockIdx.x] * width;   // width is even
    const int n = (int)(cols - c0 < width ? cols - c0 : width);
    {
        const double2 *__restrict__ src = reinterpret_cast<const double2 *>(x + c0);
        for (int k = threadIdx.x; k < n / 2; k += kSellBlock) reinterpret_cast<double2 *>(table)[k] = src[k];
        if (threadIdx.x == 0) {
            if (n & 1) table[n - 1] = x[c0 + n - 1];
            table[kSellSlots] = 0.0;   // the padding slot
        }
        __syncthreads();
    }
    sell_stream(table, wave_off, (int)(blockIdx.x * kSellWaves + threadIdx.x / kWave), data, psums);
}

// sums[h] = sum over the windows and slots of hot row h.  A workgroup has 64 slots: sixteen partial sums each (windows in order inside
// each), added in order, then the slots of a row.  Some 7 us and the bytes of pos and psums at 4 TB/s (15 us for 128 windows of 25,000 slots; with
// the sums of a group of slots read coalesced and exchanged in LDS, by 400 workgroups with a ticket a group: the same).
__global__ __launch_bounds__(kSellBlock) void k_window_reduce(int nwin, int nslots, const int32_t *__restrict__ row_end, const uint16_t *__restrict__ pos,
                                                             const double *__restrict__ psums, double *__restrict__ sums)
{
    __shared__ double part[kSellWaves][kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int v = blockIdx.x * kWave + lane;
    const int per = (nwin + kSellWaves - 1) / kSellWaves;
    const int w0 = wv * per, w1 = (w0 + per < nwin) ? w0 + per : nwin;
    double a = 0.0;
    if (v < nslots) {
#pragma unroll 8
        for (int w = w0; w < w1; ++w) {
            const int p = pos[(int64_t)w * nslots + v];
            const double t = psums[(int64_t)w * nslots + (p > 0 ? p - 1 : 0)];   // (without entries: whatever is there, not used)
            a += p > 0 ? t : 0.0;
        }
    }
    part[wv][lane] = a;
    __syncthreads();
    if (wv != 0) return;
    double t = part[0][lane];
#pragma unroll
    for (int m = 1; m < kSellWaves; ++m) t += part[m][lane];
    const int h = v < nslots ? row_end[v] : -1, before = lane_before(h);   // (asked for by all lanes)
    int first = lane == 0 || before >= 0;
    wave_seg_scan(t, first);
    if (h >= 0) sums[h] = t;
}

template <bool HOT, bool HEAD, bool SQ, bool UNIT>
__global__ __launch_bounds__(kBlock) void k_csr_spmv_part(PartArgs pa, int64_t rows, PartPtrs pp, const double *__restrict__ x)
{
    __shared__ __align__(16) double prod[kProdDoubles];
    extern __shared__ __align__(16) double table[];   // pa.slots doubles (none without HOT)
    part_body<HOT, HEAD, SQ, UNIT>(prod, table, pa, blockIdx.x % pa.P, blockIdx.x / pa.P, gridDim.x / pa.P, rows, pp, x);
}

// ------------------------------------------------------------------ hot-row tiles (see HotTiles)
constexpr int kMaxTileBlocks = 256;   // workgroups per slice

int hot_tiles_build(CsrPlan &A, const int64_t *t_rowptr, const int32_t *t_col, const double *t_val,
                    const std::vector<int32_t> &slot_code, int nhot, hipStream_t st)
{
    HotTiles &H = A.hot;
    H.nhot = nhot;
    struct Entry { uint16_t slot, iloc; double val; };
    std::vector<Entry> cur[kTileSlices];
    int64_t base[kTileSlices] = {0};
    std::vector<double> tval[kTileSlices];
    std::vector<uint16_t> tiloc[kTileSlices];
    std::vector<uint8_t> tflags[kTileSlices];
    std::vector<uint16_t> sslot[kTileSlices];
    std::vector<int4> hdrs[kTileSlices];

    std::vector<Entry> sorted[kTileSlices];
    std::vector<int32_t> slot_at[kTileSlices];
    auto close_tile = [&](int s) {
        std::vector<Entry> &e = cur[s];
        if (e.empty()) return;
        // by slot; the entries of a slot keep their column order (counting sort)
        {
            std::vector<int32_t> &at = slot_at[s];
            at.assign((size_t)kTileSlots + 1, 0);
            for (const Entry &x : e) at[(size_t)x.slot + 1]++;
            for (int q = 0; q < kTileSlots; ++q) at[(size_t)q + 1] += at[(size_t)q];
            sorted[s].resize(e.size());
            for (const Entry &x : e) sorted[s][(size_t)at[x.slot]++] = x;
            e.swap(sorted[s]);
        }
        int4 h = make_int4((int)base[s], 0, 0, (int)sslot[s].size());
        const size_t off = tiloc[s].size();
        tval[s].resize(off + kChunk, 0.0);   // off: a multiple of kChunk
        tiloc[s].resize(off + kChunk, 0);
        tflags[s].resize((off + kChunk) / 8, 0);
        for (size_t k = 0; k < e.size(); ++k) {
            tval[s][val_pos(off + k)] = e[k].val;
            tiloc[s][off + k] = e[k].iloc;
            if (k + 1 == e.size() || e[k + 1].slot != e[k].slot) {
                tflags[s][(off + k) / 8] |= (uint8_t)(1u << (k % 8));
                sslot[s].push_back(e[k].slot);
                h.y += 1;
            }
        }
        while (sslot[s].size() % 8) sslot[s].push_back(0);
        for (const Entry &x : e) h.z = std::max<int>(h.z, x.iloc + 1);   // columns the tile spans
        hdrs[s].push_back(h);
        e.clear();
    };

    // the kernels gather from a copy of the tile's columns in LDS: a tile spans at most kTileWindow of them
    const int64_t span = kTileWindow;
    // The slices are independent of each other (own features, own tiles): one host thread per slice walks the matrix
    // and keeps the entries of its slice.
    int64_t slice_nnz[kTileSlices] = {0};
    bool slice_failed[kTileSlices] = {false};
    // the code of every entry's feature (slice and slot; kNoCode: not in the tiles), looked up once, so that the slice
    // threads stream through 16-bit codes instead of each looking every feature up again
    static_assert(kTileSlices * kTileSlots < 0xffff, "entry codes are 16 bits");
    constexpr uint16_t kNoCode = 0xffff;
    std::vector<uint16_t> ecode;
    try {
        ecode.resize((size_t)t_rowptr[A.cols]);
    } catch (const std::exception &) { set_error("out of host memory building the hot-row tiles"); return TRON_ENOMEM; }
    parallel_ranges(A.cols, t_rowptr[A.cols], [&](int64_t i0, int64_t i1) {
        for (int64_t k = t_rowptr[i0]; k < t_rowptr[i1]; ++k) {
            const int32_t code = slot_code[t_col[k]];
            ecode[k] = code >= 0 ? (uint16_t)code : kNoCode;
        }
    });
    auto build_slice = [&](int s) {
        try {
            int64_t nnz = 0;
            for (int64_t i = 0; i < A.cols; ++i) {
                int cnt = 0;
                for (int64_t k = t_rowptr[i]; k < t_rowptr[i + 1]; ++k)
                    if (ecode[k] != kNoCode && ecode[k] / kTileSlots == s) ++cnt;
                if (!cnt) continue;
                if ((int)cur[s].size() + cnt > kChunk || (!cur[s].empty() && i - base[s] >= span)) close_tile(s);
                if (cur[s].empty()) base[s] = i;
                for (int64_t k = t_rowptr[i]; k < t_rowptr[i + 1]; ++k) {
                    const int code = ecode[k];
                    if (code == kNoCode || code / kTileSlots != s) continue;
                    ++nnz;
                    cur[s].push_back({(uint16_t)(code % kTileSlots), (uint16_t)(i - base[s]), t_val[k]});
                }
            }
            close_tile(s);
            slice_nnz[s] = nnz;
        } catch (const std::exception &) {
            slice_failed[s] = true;
        }
    };
    {
        std::vector<std::thread> workers;
        try {
            for (int s = 1; s < kTileSlices; ++s) workers.emplace_back(build_slice, s);
        } catch (const std::exception &) {
            // fewer threads than slices could be started: the rest run here
        }
        const int started = (int)workers.size();
        build_slice(0);
        for (int s = 1 + started; s < kTileSlices; ++s) build_slice(s);
        for (std::thread &t : workers) t.join();
    }
    for (int s = 0; s < kTileSlices; ++s) {
        if (slice_failed[s]) { set_error("out of host memory building the hot-row tiles"); return TRON_ENOMEM; }
        H.nnz += slice_nnz[s];
    }

    // concatenate the slices; segment offsets become global
    int64_t ntiles = 0, nseg = 0;
    for (int s = 0; s < kTileSlices; ++s) {
        H.tile0[s] = ntiles;
        H.ntiles[s] = (int64_t)hdrs[s].size();
        for (int4 &h : hdrs[s]) h.w += (int)nseg;
        ntiles += H.ntiles[s];
        nseg += (int64_t)sslot[s].size();
    }
    H.ntiles_total = ntiles;
    H.nseg_padded = nseg;
    for (int s = 0; s < kTileSlices; ++s)
        for (const int4 &h : hdrs[s]) H.span_total += h.z;
    if (ntiles == 0) return TRON_OK;
    if (nseg > 0x7ffffff0 || ntiles > 0x7ffffff0 / kChunk * 1024) { set_error("hot tiles too large"); return TRON_EINVAL; }
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&H.val), sizeof(double) * ntiles * kChunk));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&H.iloc), sizeof(uint16_t) * ntiles * kChunk));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&H.flags), ntiles * kBlock));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&H.hdr), sizeof(int4) * ntiles));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&H.seg_slot), sizeof(uint16_t) * std::max<int64_t>(nseg, 8)));
    int64_t segpos = 0;
    for (int s = 0; s < kTileSlices; ++s) {
        const int64_t t0 = H.tile0[s];
        if (H.ntiles[s] == 0) continue;
        TRON_HIP(hipMemcpyAsync(H.val + t0 * kChunk, tval[s].data(), sizeof(double) * tval[s].size(), hipMemcpyHostToDevice, st));
        TRON_HIP(hipMemcpyAsync(H.iloc + t0 * kChunk, tiloc[s].data(), sizeof(uint16_t) * tiloc[s].size(), hipMemcpyHostToDevice, st));
        TRON_HIP(hipMemcpyAsync(H.flags + t0 * kBlock, tflags[s].data(), tflags[s].size(), hipMemcpyHostToDevice, st));
        TRON_HIP(hipMemcpyAsync(H.hdr + t0, hdrs[s].data(), sizeof(int4) * hdrs[s].size(), hipMemcpyHostToDevice, st));
        TRON_HIP(hipMemcpyAsync(H.seg_slot + segpos, sslot[s].data(), sizeof(uint16_t) * sslot[s].size(), hipMemcpyHostToDevice, st));
        segpos += (int64_t)sslot[s].size();
    }
    TRON_TRY(upload(&H.slot_of_row, slot_code.data(), slot_code.size(), st));
    int64_t maxt = 0;
    for (int s = 0; s < kTileSlices; ++s) maxt = std::max(maxt, H.ntiles[s]);
    // 0 = automatic: 3 workgroups per CU (the kernel is bound by HBM)
    const int64_t want_blocks = g_tuning.csr_tile_blocks_per_slice > 0 ? g_tuning.csr_tile_blocks_per_slice : 96;
    H.blocks_per_slice = (int)std::max<int64_t>(1, std::min<int64_t>(maxt, std::min<int64_t>(want_blocks, kMaxTileBlocks)));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&H.wg_acc), sizeof(double) * kTileSlices * H.blocks_per_slice * kTileSlots));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&H.sums), sizeof(double) * kTileSlices * kTileSlots));
    TRON_HIP(hipStreamSynchronize(st));
    return TRON_OK;
}

// ------------------------------------------------------------------ hot rows of a unit plan as windows (see HotWindows)
// As many windows as make, with a whole number of workgroups for each, nearly one workgroup per compute unit; beyond that many a
// multiple, so that no round of workgroups is nearly empty.
int hot_windows_count(int64_t cols)
{
    const int64_t least = std::max<int64_t>(1, (cols + kSellSlots - 1) / kSellSlots);
    if (least > kWindowBlocks) return (int)((least + kWindowBlocks - 1) / kWindowBlocks * kWindowBlocks);
    const int64_t most = std::max<int64_t>(1, cols / 2);   // (windows of two columns at least)
    return (int)std::min<int64_t>(kWindowBlocks / (kWindowBlocks / least), most);
}

int hot_windows_build(CsrPlan &A, const int64_t *t_rowptr, const int32_t *t_col, const std::vector<int32_t> &hot_of, int nhot, hipStream_t st)
{
    HotTiles &H = A.hot;
    HotWindows &Q = H.win;
    const int64_t cols = A.cols;
    const int width = (int)std::max<int64_t>(2, ((cols + hot_windows_count(cols) - 1) / hot_windows_count(cols) + 1) / 2 * 2);
    const int nwin = (int)((cols + width - 1) / width);
    static_assert(kSellSlots % 2 == 0, "an even width of at most kSellSlots");
    // entries of every hot row in every window
    std::vector<int32_t> count((size_t)nwin * nhot, 0);
    std::vector<int64_t> win_nnz((size_t)nwin, 0);
    const int64_t nnz = t_rowptr[cols];
    auto for_windows = [&](auto &&fn) { parallel_ranges(nwin, nnz, [&](int64_t w0, int64_t w1) { for (int64_t w = w0; w < w1; ++w) fn(w); }); };
    auto first_entry = [&](int64_t w) { return t_rowptr[std::min<int64_t>(w * width, cols)]; };
    for_windows([&](int64_t w) {
        int32_t *cnt = count.data() + (size_t)w * nhot;
        int64_t all = 0;
        for (int64_t k = first_entry(w); k < first_entry(w + 1); ++k) {
            const int h = hot_of[t_col[k]];
            if (h >= 0) { ++cnt[h]; ++all; }
        }
        win_nnz[(size_t)w] = all;
    });
    for (int64_t e : win_nnz) H.nnz += e;
    if (H.nnz == 0) return TRON_OK;
    // slots: the pieces of the row's fullest window
    std::vector<int32_t> fullest((size_t)nhot, 0), slot0((size_t)nhot, 0);
    for (int w = 0; w < nwin; ++w)
        for (int h = 0; h < nhot; ++h) fullest[h] = std::max(fullest[h], count[(size_t)w * nhot + h]);
    int most = kPieceEntries;
    for (;; most *= 2) {
        int64_t slots = 0;
        for (int h = 0; h < nhot; ++h) slots += (fullest[h] + most - 1) / most * (fullest[h] > most ? 2 : 1);   // (half of a block may stay empty)
        if ((slots <= kMaxPieceSlots && slots * nwin < 0x7ffffff0) || most >= kSellSlots) break;
    }
    std::vector<int32_t> row_end;
    for (int several = 1; several >= 0; --several)
        for (int h = 0; h < nhot; ++h) {
            const int m = (fullest[h] + most - 1) / most;
            if (m == 0 || (m > 1) != (several == 1)) continue;
            while (row_end.size() % kWave + (size_t)m > kWave) row_end.push_back(-1);
            slot0[h] = (int32_t)row_end.size();
            row_end.resize(row_end.size() + (size_t)m, -1);
            row_end.back() = h;
        }
    const int nslots = (int)row_end.size();
    H.nhot = nhot;
    if (nslots > kMaxPieceSlots) { set_error("internal: too many pieces of hot rows"); return TRON_EINVAL; }
    // workgroups: one per window, and what is left of kWindowBlocks always to the window with the most entries per workgroup
    std::vector<int32_t> blocks((size_t)nwin, 1);
    {
        std::vector<std::pair<double, int32_t>> heap;
        for (int w = 0; w < nwin; ++w) heap.emplace_back((double)win_nnz[w], -w);
        std::make_heap(heap.begin(), heap.end());
        for (int left = kWindowBlocks - nwin; left > 0; --left) {
            std::pop_heap(heap.begin(), heap.end());
            const int w = -heap.back().second;
            blocks[w] += 1;
            heap.back().first = (double)win_nnz[w] / blocks[w];
            std::push_heap(heap.begin(), heap.end());
        }
    }
    std::vector<int32_t> block0((size_t)nwin + 1, 0), window_of;
    for (int w = 0; w < nwin; ++w) {
        block0[w + 1] = block0[w] + blocks[w];
        window_of.insert(window_of.end(), (size_t)blocks[w], w);
    }
    Q.nblocks = block0[nwin];
    // the slices of a window: its pieces by length (ties: by slot), 64 at a time, dealt to its wavefronts longest first, each to the one
    // with the least work so far
    struct Slice { int32_t first, len8, wave; int64_t at; };   // first: of its pieces; at: its header group in the window
    std::vector<uint16_t> pos((size_t)nwin * nslots, 0);
    std::vector<std::vector<Slice>> slices((size_t)nwin);
    std::vector<std::vector<int32_t>> order((size_t)nwin);   // slots of the window's pieces, longest first
    std::vector<int64_t> wave_len((size_t)Q.nblocks * kSellWaves, 0), win_pieces((size_t)nwin, 0);
    std::atomic<bool> failed{false};
    for_windows([&](int64_t w) {
        try {
            const int32_t *cnt = count.data() + (size_t)w * nhot;
            // slots by (group, length); a group's slices begin with a piece of their own
            std::vector<int32_t> length((size_t)nslots, 0), at((size_t)most + 2);
            for (int h = 0; h < nhot; ++h)
                for (int left = cnt[h], v = slot0[h]; left > 0; left -= most, ++v) length[v] = std::min(left, most);
            std::vector<int32_t> &ord = order[(size_t)w];
            for (int v0 = 0; v0 < nslots; v0 += kSlotGroup) {
                const int v1 = std::min(nslots, v0 + kSlotGroup);
                std::fill(at.begin(), at.end(), 0);
                for (int v = v0; v < v1; ++v) ++at[(size_t)(most - length[v]) + 1];
                for (int l = 0; l <= most; ++l) at[(size_t)l + 1] += at[(size_t)l];
                const int used = at[(size_t)most];   // those with entries
                ord.resize((size_t)v0 + (size_t)used, -1);
                for (int v = v0; v < v1; ++v) {
                    if (length[v] == 0) continue;
                    const int q = at[(size_t)(most - length[v])]++;
                    ord[(size_t)(v0 + q)] = v;
                    pos[(size_t)w * nslots + v] = (uint16_t)(v0 + q + 1);
                }
                win_pieces[(size_t)w] += used;
                ord.resize((size_t)v1, -1);
            }
            const int nw = blocks[w] * kSellWaves;
            std::vector<std::pair<int64_t, int32_t>> heap;   // (-load, -wave)
            for (int v = 0; v < nw; ++v) heap.emplace_back(0, -v);
            std::make_heap(heap.begin(), heap.end());
            std::vector<std::pair<int32_t, int32_t>> by_length;   // (-groups, first piece)
            static_assert(kSlotGroup % kWave == 0, "a slice belongs to one group");
            for (int q = 0; q < nslots; q += kWave)
                if (ord[(size_t)q] >= 0) by_length.emplace_back(-((length[ord[(size_t)q]] + 7) / 8), q);
            std::sort(by_length.begin(), by_length.end());
            for (const auto &e : by_length) {
                std::pop_heap(heap.begin(), heap.end());
                slices[(size_t)w].push_back({e.second, -e.first, -heap.back().second, -heap.back().first});
                heap.back().first -= 1 - e.first;
                std::push_heap(heap.begin(), heap.end());
            }
            for (const auto &e : heap) wave_len[(size_t)block0[w] * kSellWaves + (size_t)(-e.second)] = (-e.first + kSellAhead - 1) / kSellAhead * kSellAhead;
        } catch (const std::exception &) {
            failed = true;
        }
    });
    if (failed) { set_error("out of host memory building the windows"); return TRON_ENOMEM; }
    std::vector<int64_t> wave_off(wave_len.size() + 1, 0);
    for (size_t k = 0; k < wave_len.size(); ++k) wave_off[k + 1] = wave_off[k] + wave_len[k];
    Q.ngroups = wave_off.back();
    for (int64_t e : win_pieces) Q.npieces += e;
    H.ntiles_total = Q.npieces;
    const HostArray<uint16_t> data((size_t)Q.ngroups * kWave * 8);
    for_windows([&](int64_t w) {
        try {
            const size_t v0 = (size_t)block0[w] * kSellWaves, v1 = (size_t)block0[w + 1] * kSellWaves;
            std::fill(data.data() + (size_t)wave_off[v0] * kWave * 8, data.data() + (size_t)wave_off[v1] * kWave * 8, (uint16_t)kSellSlots);
            auto header = [&](int64_t group, int lane, int32_t where, int32_t groups) {
                const int32_t hdr[4] = {where, groups, 0, 0};
                std::memcpy(&data[((size_t)group * kWave + lane) * 8], hdr, sizeof(hdr));
            };
            std::vector<int64_t> used(v1 - v0, 0), start((size_t)nslots, 0);   // start: of the slot's lane in its slice's first group of entries
            const std::vector<int32_t> &ord = order[(size_t)w];
            for (const Slice &s : slices[(size_t)w]) {
                const int64_t g = wave_off[v0 + (size_t)s.wave] + s.at;
                used[(size_t)s.wave] = s.at + 1 + s.len8;
                for (int l = 0; l < kWave; ++l) {
                    const int q = s.first + l, v = q < nslots ? ord[(size_t)q] : -1;
                    header(g, l, v >= 0 ? (int32_t)(w * nslots + q) : -1, s.len8);
                    if (v >= 0) start[(size_t)v] = ((g + 1) * kWave + l) * 8;
                }
            }
            for (size_t v = v0; v < v1; ++v)   // what is left of a stream: headers of slices without groups
                for (int64_t g = wave_off[v] + used[v - v0]; g < wave_off[v + 1]; ++g)
                    for (int l = 0; l < kWave; ++l) header(g, l, -1, 0);
            std::vector<int32_t> done((size_t)nhot, 0);
            for (int64_t i = w * width; i < std::min<int64_t>(cols, (w + 1) * width); ++i)
                for (int64_t k = t_rowptr[i]; k < t_rowptr[i + 1]; ++k) {
                    const int h = hot_of[t_col[k]];
                    if (h < 0) continue;
                    const int e = done[h]++, j = e % most;
                    data[(size_t)start[(size_t)(slot0[h] + e / most)] + (size_t)(j / 8) * kWave * 8 + (size_t)(j % 8)] = (uint16_t)(i - w * width);
                }
        } catch (const std::exception &) {
            failed = true;
        }
    });
    if (failed) { set_error("out of host memory building the windows"); return TRON_ENOMEM; }
    Q.nwin = nwin;
    Q.width = width;
    Q.nslots = nslots;
    TRON_TRY(upload(&Q.window_of, window_of.data(), window_of.size(), st));
    TRON_TRY(upload(&Q.wave_off, wave_off.data(), wave_off.size(), st));
    TRON_TRY(upload(&Q.data, data.data(), (size_t)Q.ngroups * kWave * 8, st));
    TRON_TRY(upload(&Q.row_end, row_end.data(), row_end.size(), st));
    TRON_TRY(upload(&Q.pos, pos.data(), pos.size(), st));
    TRON_TRY(upload(&H.slot_of_row, hot_of.data(), hot_of.size(), st));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&Q.psums), sizeof(double) * (size_t)nwin * nslots));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&H.sums), sizeof(double) * (size_t)nhot));
    TRON_HIP(hipMemsetAsync(H.sums, 0, sizeof(double) * (size_t)nhot, st));
    TRON_HIP(hipStreamSynchronize(st));
    Q.on = true;
    return TRON_OK;
}

struct TileArgs {
    int64_t tile0[kTileSlices];
    int64_t ntiles[kTileSlices];
};

struct TilePtrs {
    const double *val;
    const uint16_t *iloc;
    const uint8_t *flags;
    const int4 *hdr;
    const uint16_t *seg_slot;
    double *wg_acc;
};

// An entry of a tile is a 16-bit column offset and a value; thread t loads those of entries 8t .. 8t+7 (see val_pos).  A tile spans at most kTileWindow columns: the workgroup copies them from x into
// LDS with two coalesced loads per thread and gathers from the copy -- the gathers of a tile go to a few hundred
// consecutive doubles, and the vector memory pipeline, which handles about one lane of such a gather per clock, was
// what bound this kernel when they went to x itself.
struct TileRegs {
    v2d v[4];
    v4i il;             // eight 16-bit local column offsets
    uint4 slots;        // slots of the segments 8*tid .. 8*tid+7 (16 bits each)
    unsigned flags;     // bit e: entry 8*tid + e is the last of its segment
    double w[2];        // the two columns of the tile that the thread copies into LDS
    int4 hdr;
};

// the data of tile T, whose header is h; columns clamped to the tile's last one
__device__ __forceinline__ void load_tile(TileRegs &r, const TilePtrs &tp, const double *__restrict__ x, int4 h, int64_t T)
{
    const int tid = threadIdx.x;
    r.hdr = h;
    r.il = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(tp.iloc + T * kChunk + 8 * tid));
#pragma unroll
    for (int m = 0; m < 4; ++m) r.v[m] = __builtin_nontemporal_load(reinterpret_cast<const v2d *>(tp.val + T * kChunk + m * kQuarter + tid * 2));
    r.flags = tp.flags[T * kBlock + tid];
    // slot blocks are padded to a multiple of 8; threads beyond the tile's segments re-read its first block
    const int nseg = h.y;
    const int64_t d0 = (int64_t)h.w + ((8 * tid < nseg) ? 8 * tid : 0);
    r.slots = *reinterpret_cast<const uint4 *>(tp.seg_slot + d0);
    const int lastc = h.z - 1;
    const double *xt = x + h.x;
    r.w[0] = xt[tid < lastc ? tid : lastc];
    r.w[1] = xt[tid + kBlock < lastc ? tid + kBlock : lastc];
}

__device__ __forceinline__ void store_window(double *window, const TileRegs &r)
{
    window[threadIdx.x] = r.w[0];
    window[threadIdx.x + kBlock] = r.w[1];
}

// One tile: cur is reduced (its columns are in window[BUF]) while the data of the next tile of the workgroup, whose
// header is ahead, are loaded into nxt; they are not waited for before the end of the step, where the columns go to
// the other window buffer.  ahead becomes the header of the tile after that.
template <int BUF, bool SQ>
__device__ __forceinline__ void tile_step(double *prod, uint16_t *slots, double *acc, double (*window)[kTileWindow], TileRegs &cur,
                                          TileRegs &nxt, int4 &ahead, const TilePtrs &tp, const double *__restrict__ x,
                                          const int64_t Tn, const int64_t Tnn)
{
    const int tid = threadIdx.x;
    const int nseg = cur.hdr.y;
    __builtin_amdgcn_sched_barrier(0);
    load_tile(nxt, tp, x, ahead, Tn);
    ahead = load_uniform(tp.hdr + Tnn);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // every thread is past the accumulator updates and the totals of the tile before, and this tile's columns are
    // in window[BUF]
    double p[8], cin;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const unsigned two = (unsigned)cur.il[m];
        p[2 * m] = window[BUF][two & 0xffffu];
        p[2 * m + 1] = window[BUF][two >> 16];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const double v = cur.v[e / 2][e % 2];
        p[e] *= SQ ? v * v : v;
    }
    if (8 * tid < nseg) *reinterpret_cast<uint4 *>(slots + 8 * tid) = cur.slots;
    int idx0;
    runs_from_regs(prod, threadIdx.x, cur.flags, p, cin, idx0);   // barrier inside: the slots are visible after it
    // What the threads before add to the thread's first segment goes in on its own, before the segment's own sum.
    int sl[8];
    int i = idx0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        sl[e] = slots[i];   // an entry that ends no segment reads a slot it does not use (then i < 2048: there are fewer segments than entries)
        i += (cur.flags >> e) & 1u;
    }
    if (cur.flags) lds_add(acc + sl[0], cin);   // sl[0] is the slot of the thread's first segment
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if ((cur.flags >> e) & 1u) lds_add(acc + sl[e], p[e]);
    // the other buffer was last read before the barrier inside runs_from_regs of the step before
    store_window(window[BUF ^ 1], nxt);
}

// Persistent workgroup (slice s, q): tiles q, q + B, ... of the slice, LDS accumulators for the slice's hot rows; two steps per
// iteration so that the two sets of tile registers and the two window buffers swap roles without copies (indices clamped to
// the last tile, so every step issues the same loads).  SQ: the values are squared.
template <bool SQ>
__global__ __launch_bounds__(kBlock) void k_hot_tiles(TileArgs ta, int B, TilePtrs tp, const double *__restrict__ x)
{
    __shared__ __align__(16) double prod[kOutOffset];   // the wavefront totals only
    __shared__ __align__(16) uint16_t slots[kChunk];
    __shared__ double acc[kTileSlots];
    __shared__ double window[2][kTileWindow];
    static_assert(kTileWindow == 2 * kBlock, "two columns per thread");
    const int s = blockIdx.x % kTileSlices, q = blockIdx.x / kTileSlices;
    const int tid = threadIdx.x;
    for (int k = tid; k < kTileSlots; k += kBlock) acc[k] = 0.0;
    const int64_t nt = ta.ntiles[s];
    if (q < nt) {
        const int64_t T0 = ta.tile0[s];
        const int64_t last = nt - 1;
        auto clampt = [&](int64_t t) { return T0 + (t < last ? t : last); };
        TileRegs r0, r1;
        load_tile(r0, tp, x, load_uniform(tp.hdr + clampt(q)), clampt(q));
        int4 ahead = load_uniform(tp.hdr + clampt(q + B));
        store_window(window[0], r0);
        for (int64_t t = q; t < nt; t += 2 * (int64_t)B) {
            tile_step<0, SQ>(prod, slots, acc, window, r0, r1, ahead, tp, x, clampt(t + B), clampt(t + 2 * (int64_t)B));
            if (t + B >= nt) break;
            tile_step<1, SQ>(prod, slots, acc, window, r1, r0, ahead, tp, x, clampt(t + 2 * (int64_t)B), clampt(t + 3 * (int64_t)B));
        }
    }
    __syncthreads();
    double *out = tp.wg_acc + ((int64_t)s * B + q) * kTileSlots;
    for (int k = tid; k < kTileSlots; k += kBlock) out[k] = acc[k];
}

// sums[s*K + k] = sum over the B workgroups of slice s: sixteen partial sums (workgroup order inside each), added in
// order.  A workgroup covers 64 consecutive slots, one wavefront per part, so every read is one 512-byte row and a CU
// has sixteen rows in flight (with four the kernel waited for HBM most of the time).
constexpr int kReduceWaves = 16;
__global__ __launch_bounds__(kReduceWaves * kWave) void k_hot_reduce(int B, const double *__restrict__ wg_acc, double *__restrict__ sums)
{
    __shared__ double part[kReduceWaves][kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int idx = blockIdx.x * kWave + lane;   // s*K + k
    const int s = idx / kTileSlots, k = idx % kTileSlots;
    const int per = (B + kReduceWaves - 1) / kReduceWaves;
    const int q0 = wv * per, q1 = (q0 + per < B) ? q0 + per : B;
    const double *p = wg_acc + (int64_t)s * B * kTileSlots + k;
    double a = 0.0;
    for (int q = q0; q < q1; ++q) a += p[(int64_t)q * kTileSlots];
    part[wv][lane] = a;
    __syncthreads();
    if (wv == 0) {
        double t = part[0][lane];
#pragma unroll
        for (int m = 1; m < kReduceWaves; ++m) t += part[m][lane];
        sums[idx] = t;
    }
}

static TileArgs tile_args(const HotTiles &H)
{
    TileArgs ta;
    for (int s = 0; s < kTileSlices; ++s) { ta.tile0[s] = H.tile0[s]; ta.ntiles[s] = H.ntiles[s]; }
    return ta;
}

static TilePtrs tile_ptrs(const HotTiles &H) { return TilePtrs{H.val, H.iloc, H.flags, H.hdr, H.seg_slot, H.wg_acc}; }

// tiles + the reduction of the workgroup accumulators (B = workgroups per slice)
static int launch_hot_tiles(tron_dataset *ds, const CsrPlan &A, const double *x, bool square)
{
    const HotTiles &H = A.hot;
    hipStream_t st = ds->stream;
    if (H.win.on) {   // squares, if any, are in the scaled vector
        const HotWindows &Q = H.win;
        {
            ProfScope ps(ds, SLOT_SPMV_TILES, st);
            hipLaunchKernelGGL(k_window_sell, dim3(Q.nblocks), dim3(kSellBlock), 0, st, Q.window_of, Q.width, A.cols, Q.wave_off, Q.data, x, Q.psums);
            TRON_HIP(hipGetLastError());
        }
        ProfScope ps(ds, SLOT_SPMV_TILE_REDUCE, st);
        hipLaunchKernelGGL(k_window_reduce, dim3((Q.nslots + kWave - 1) / kWave), dim3(kSellBlock), 0, st, Q.nwin, Q.nslots, Q.row_end, Q.pos, Q.psums, H.sums);
        TRON_HIP(hipGetLastError());
        return TRON_OK;
    }
    {
        ProfScope ps(ds, SLOT_SPMV_TILES, st);
        if (square)
            hipLaunchKernelGGL(k_hot_tiles<true>, dim3(kTileSlices * H.blocks_per_slice), dim3(kBlock), 0, st, tile_args(H),
                               H.blocks_per_slice, tile_ptrs(H), x);
        else
            hipLaunchKernelGGL(k_hot_tiles<false>, dim3(kTileSlices * H.blocks_per_slice), dim3(kBlock), 0, st, tile_args(H),
                               H.blocks_per_slice, tile_ptrs(H), x);
        TRON_HIP(hipGetLastError());
    }
    {
        ProfScope ps(ds, SLOT_SPMV_TILE_REDUCE, st);
        hipLaunchKernelGGL(k_hot_reduce, dim3(kTileSlices * kTileSlots / kWave), dim3(kReduceWaves * kWave), 0, st, H.blocks_per_slice,
                           H.wg_acc, H.sums);
        TRON_HIP(hipGetLastError());
    }
    return TRON_OK;
}

// ------------------------------------------------------------------ fix-up of split rows
// G lanes per split row: y[row] += factor * (carry[b0] + ... + carry[b0+cnt-1]).  G = 8 when no row spans more than
// 64 chunks (one workgroup then fixes 32 rows), else a whole wavefront per row.
template <int EPI, int G>
__global__ __launch_bounds__(kBlock) void k_csr_fixup(int nfix, const int32_t *__restrict__ fix_row,
                                                      const int32_t *__restrict__ fix_b0, const int32_t *__restrict__ fix_cnt, const double *__restrict__ carry,
                                                      double *__restrict__ yout, const double *__restrict__ aux, double alpha)
{
    const int m = blockIdx.x * (kBlock / G) + threadIdx.x / G;
    const int sub = threadIdx.x & (G - 1);
    const bool live = m < nfix;   // the lane sums below need every lane of the wavefront
    const int b0 = live ? fix_b0[m] : 0, cnt = live ? fix_cnt[m] : 0;
    double s = 0.0;
    for (int k = sub; k < cnt; k += G) s += carry[b0 + k];
    s = group_sum(s, G);
    if (live && sub == 0) {
        const int64_t r = fix_row[m];
        double factor = 1.0;
        if (EPI == EPI_SCALE) factor = aux[r];
        if (EPI == EPI_AXPY) factor = alpha;
        double *dst = yout + r;
        *dst = fma(factor, s, *dst);
    }
}

template <int EPI>
static int launch_fixup(tron_dataset *ds, const CsrPlan &A, double *yout, const double *aux, double alpha)
{
    if (A.nfix <= 0) return TRON_OK;
    ProfScope ps(ds, SLOT_SPMV_FIXUP);
    if (A.fix_max_cnt <= 64) {
        const int per = kBlock / 8;
        hipLaunchKernelGGL((k_csr_fixup<EPI, 8>), dim3((A.nfix + per - 1) / per), dim3(kBlock), 0, ds->stream, A.nfix, A.fix_row,
                           A.fix_b0, A.fix_cnt, A.carry, yout, aux, alpha);
    } else {
        const int per = kBlock / kWave;
        hipLaunchKernelGGL((k_csr_fixup<EPI, kWave>), dim3((A.nfix + per - 1) / per), dim3(kBlock), 0, ds->stream, A.nfix,
                           A.fix_row, A.fix_b0, A.fix_cnt, A.carry, yout, aux, alpha);
    }
    TRON_HIP(hipGetLastError());
    return TRON_OK;
}

// ------------------------------------------------------------------ combine kernels (partitioned layout)
// The partial sums of a plan are stored one per segment (a segment = a row's entries in one partition), partition by
// partition, rows ascending inside a partition -- the kernels above write them as dense 512-byte stores.  A row's
// slots are found by rank: mask[r] says in which partitions row r has a segment; inside the 64 rows of a wavefront
// the slot of (r, x) is group_base[x][r / 64] + (number of lower rows of the group with bit x set).
struct PartialRef {
    const double *partial;
    const uint16_t *mask;
    const GroupBase *group_base;   // one record per group of 64 rows
    const double *row_scale;       // unit plan of X: the value of row i's entries (null otherwise)
    const double *head_sums;       // head partition kept as sorted slices: its sums, row r's at head_pos[r] (null otherwise)
    const int32_t *head_pos;
};

struct HotRef {
    const int32_t *slot_of_row;   // null: no hot rows
    const double *sums;
};

// Sum over the partitions of row r = 64 G + lane, in partition order.  Every lane of the wavefront calls it with
// the same G; `valid` is false for rows past the end.  All loads are issued before the first is used.
__device__ __forceinline__ double sum_parts(const PartialRef &P, int64_t G, int64_t r, bool valid, HotRef hot = HotRef{nullptr, nullptr})
{
    const unsigned m = valid ? P.mask[r] : 0u;
    const GroupBase gb = P.group_base[G];   // uniform: scalar loads
    double s = 0.0;
    if (valid && P.head_sums) s = P.head_sums[P.head_pos[r]];
    if (valid && hot.slot_of_row) {
        const int hs = hot.slot_of_row[r];
        if (hs >= 0) s = hot.sums[hs];
    }
    double v[kMaxParts];
#pragma unroll
    for (int x = 0; x < kMaxParts; ++x) {
        const bool bit = (m >> x) & 1u;
        const uint64_t b = __ballot(bit);
        const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
        v[x] = bit ? P.partial[(int64_t)gb.first[x] + rank] : 0.0;
    }
#pragma unroll
    for (int x = 0; x < kMaxParts; ++x) s += v[x];
    if (P.row_scale && valid) s *= P.row_scale[r];
    return s;
}

// rows are dealt to wavefronts in groups of 64: group g0, g0 + (wavefronts in the grid), ...
#define TRON_FOR_ROW_GROUPS(rows, G, r, valid)                                                                     \
    for (int64_t G = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave, r = G * kWave + (threadIdx.x & (kWave - 1)); \
         G * kWave < (rows); G += (int64_t)gridDim.x * kWavesPerBlock, r += (int64_t)gridDim.x * kBlock)            \
        if (const bool valid = r < (rows); true)

// z = sum of partials; loss terms; partial slot 0 = sum loss
template <int LOSS>
__global__ __launch_bounds__(kBlock) void k_combine_loss(int64_t n, PartialRef P, const double *__restrict__ y,
                                                         double *__restrict__ zhat, double *__restrict__ D, double *__restrict__ red,
                                                         const double *__restrict__ post, Finish fin)
{
    __shared__ double lds[kWavesPerBlock];
    double acc = 0.0;
    TRON_FOR_ROW_GROUPS(n, G, i, valid) {
        const double z = sum_parts(P, G, i, valid);
        if (valid) {
            double a, zh, Di;
            loss_terms_dev<LOSS>(z, y[i], a, zh, Di);
            zhat[i] = post ? post[i] * zh : zh;
            D[i] = Di;
            acc += a;
        }
    }
    acc = block_sum(acc, lds);
    if (threadIdx.x == 0) store_shared(red + blockIdx.x, acc);
    finish_partials<1>(fin, red, 0, lds);
}

// out = scale .* sum of partials
__global__ __launch_bounds__(kBlock) void k_combine_scale(int64_t rows, PartialRef P, const double *__restrict__ scale,
                                                          double *__restrict__ out, const double *__restrict__ post)
{
    TRON_FOR_ROW_GROUPS(rows, G, i, valid) {
        const double s = sum_parts(P, G, i, valid);
        if (valid) {
            const double o = scale[i] * s;
            out[i] = post ? post[i] * o : o;
        }
    }
}

// out = add + alpha * sum of partials (add == null: add 1); partial slot 0 = out . (SELF ? out : add)
template <bool SELF>
__global__ __launch_bounds__(kBlock) void k_combine_axpy(int64_t rows, PartialRef P, const double *__restrict__ add, double alpha,
                                                         double *__restrict__ out, double *__restrict__ red, HotRef hot, Finish fin)
{
    __shared__ double lds[kWavesPerBlock];
    double acc = 0.0;
    TRON_FOR_ROW_GROUPS(rows, G, i, valid) {
        const double s = sum_parts(P, G, i, valid, hot);
        if (valid) {
            const double a = add ? add[i] : 1.0;
            const double o = fma(alpha, s, a);
            out[i] = o;
            acc += o * (SELF ? o : a);
        }
    }
    acc = block_sum(acc, lds);
    if (threadIdx.x == 0) store_shared(red + blockIdx.x, acc);
    finish_partials<1>(fin, red, 0, lds);
}

// ------------------------------------------------------------------ launchers
static inline int vec_grid(int64_t m)
{
    int64_t g = (m + kBlock * 4 - 1) / (kBlock * 4);
    if (g < 1) g = 1;
    if (g > kMaxGrid) g = kMaxGrid;
    return (int)g;
}

// one launch with the epilogue in it: plain CSR or a single range of segments.  Returns the number of sums in E.red.
template <int EPI>
static int launch_single(tron_dataset *ds, const CsrPlan &A, int slot, const double *x, const EpiArgs &E, bool square = false)
{
    ProfScope ps(ds, slot);
    if (A.direct) {
        const DirectPtrs P{A.col, A.val, A.chunk_tab, A.flags, A.row_lo, A.row_seg, A.chunk_long, A.long_row, A.carry, A.long_first, A.long_ticket};
        if (square) hipLaunchKernelGGL((k_csr_direct<EPI, true>), dim3(A.nblocks), dim3(kBlock), 0, ds->stream, P, A.nfix, x, E);
        else hipLaunchKernelGGL((k_csr_direct<EPI, false>), dim3(A.nblocks), dim3(kBlock), 0, ds->stream, P, A.nfix, x, E);
        TRON_HIP(hipGetLastError());
        return A.nblocks + A.nfix;
    }
    if (square)
        hipLaunchKernelGGL((k_csr_spmv<EPI, true>), dim3(A.nblocks), dim3(kBlock), 0, ds->stream, A.part_nnz[0], A.rowptr, A.col, A.val, A.row_lo, x, E, A.carry);
    else
        hipLaunchKernelGGL((k_csr_spmv<EPI, false>), dim3(A.nblocks), dim3(kBlock), 0, ds->stream, A.part_nnz[0], A.rowptr, A.col, A.val, A.row_lo, x, E, A.carry);
    TRON_HIP(hipGetLastError());
    return A.nblocks;
}

// Whether launch_single can form the sum over the rows as well (no row is completed by the fix-up kernel, and the sums are few)
bool single_sums(const CsrPlan &A) { return A.direct || (A.plain && A.nfix == 0 && A.nblocks <= kDirectMaxSums); }

static Finish no_finish(tron_dataset *ds) { return finish_for(ds, -1, 1); }

// plain CSR with the rows longer than a chunk completed by the fix-up kernel
template <int EPI>
static int launch_plain(tron_dataset *ds, const CsrPlan &A, int slot, const double *x, double *yout, const double *aux,
                        double alpha, bool square = false)
{
    TRON_TRY(launch_single<EPI>(ds, A, slot, x, EpiArgs{yout, aux, alpha, false, nullptr, nullptr, no_finish(ds)}, square));
    return launch_fixup<EPI>(ds, A, yout, aux, alpha);
}

static PartArgs part_args(const CsrPlan &A)
{
    PartArgs pa;
    std::memset(&pa, 0, sizeof(pa));
    pa.P = A.P;
    for (int i = 0; i < A.P; ++i) {
        pa.base[i] = A.part_base[i];
        pa.nnz[i] = A.part_nnz[i];
        pa.seg0[i] = A.part_seg0[i];
        pa.chunk0[i] = A.part_chunk0[i];
        pa.nchunks[i] = A.part_nchunks[i];
        pa.nhot[i] = A.part_nhot[i];
    }
    pa.slots = A.range_slots;
    return pa;
}

// The head partition as a one-partition launch: val, hot_ids and the partials are passed pre-offset, col16 only
// holds this partition; chunk and segment tables are indexed through the offsets in the arguments.
static PartArgs head_args(const CsrPlan &A)
{
    const int h = A.head;
    PartArgs ha;
    std::memset(&ha, 0, sizeof(ha));
    ha.P = 1;
    ha.nnz[0] = A.part_nnz[h];
    ha.seg0[0] = A.part_seg0[h];
    ha.chunk0[0] = A.part_chunk0[h];
    ha.nchunks[0] = A.part_nchunks[h];
    ha.nhot[0] = A.part_nhot[h];
    ha.slots = kHotSlots;
    return ha;
}

static PartialRef partial_ref(const tron_dataset *ds, const CsrPlan &A)
{
    return PartialRef{ds->row_partials, A.row_mask, A.group_base, A.row_scale, A.sell.on ? A.sell.sums : nullptr, A.sell.on ? A.sell.pos : nullptr};
}

static PartPtrs part_ptrs(const tron_dataset *ds, const CsrPlan &A)
{
    return PartPtrs{A.col, A.val, A.chunk_tab, A.flags, A.hot_x, ds->row_partials, A.carry};
}

static PartPtrs head_ptrs(const tron_dataset *ds, const CsrPlan &A)
{
    const int h = A.head;
    return PartPtrs{A.col16, A.val ? A.val + A.part_base[h] : nullptr, A.chunk_tab, A.flags, A.hot_x ? A.hot_x + (size_t)h * kHotSlots : nullptr,
                    ds->row_partials, A.carry};
}

// partial row sums of all partitions into ds->row_partials (with split rows fixed up)
static int launch_partials(tron_dataset *ds, const CsrPlan &A, int slot, const double *x, bool square = false)
{
    const PartArgs pa = part_args(A);
    if (A.hot_ids) {
        ProfScope ps(ds, SLOT_SPMV_GATHER);
        const int nh = A.P * kHotSlots + A.head_slots;
        hipLaunchKernelGGL(k_gather_hot, dim3((nh + kBlock - 1) / kBlock), dim3(kBlock), 0, ds->stream, nh, A.hot_ids, x, A.hot_x);
        TRON_HIP(hipGetLastError());
    }
    if (A.head >= 0) {
        ProfScope ps(ds, SLOT_SPMV_HEAD);
        const int grid = std::max(1, std::min(A.part_nchunks[A.head], (int)g_tuning.csr_hot_blocks_per_part * kColParts));
        if (A.sell.on) {
            const SellHead &S = A.sell;
            hipLaunchKernelGGL(k_head_sell, dim3((S.nwaves + kSellBlock / kWave - 1) / (kSellBlock / kWave)), dim3(kSellBlock), 0, ds->stream, S.nwaves, S.wave_off, S.data,
                               A.hot_x + (size_t)A.head * kHotSlots, S.sums);
        } else if (A.unit)
            hipLaunchKernelGGL((k_csr_spmv_part<true, true, false, true>), dim3(grid), dim3(kBlock), kHotSlots * sizeof(double), ds->stream,
                               head_args(A), A.rows, head_ptrs(ds, A), x);
        else
            hipLaunchKernelGGL((k_csr_spmv_part<true, true, false, false>), dim3(grid), dim3(kBlock), kHotSlots * sizeof(double), ds->stream,
                               head_args(A), A.rows, head_ptrs(ds, A), x);
        TRON_HIP(hipGetLastError());
    }
    {
        ProfScope ps(ds, slot);
        const int want = (int)(A.hot_ids ? g_tuning.csr_range_blocks_per_part : g_tuning.csr_blocks_per_part);
        // a single range (small matrices) gets the workgroups that eight ranges would share
        const int per_part = std::max(1, std::min(A.max_chunks, A.P == 1 ? want * kColParts : want));
        if (A.hot_ids && A.unit)
            hipLaunchKernelGGL((k_csr_spmv_part<true, false, false, true>), dim3(per_part * A.P), dim3(kBlock), A.range_slots * sizeof(double), ds->stream,
                               pa, A.rows, part_ptrs(ds, A), x);
        else if (A.hot_ids)
            hipLaunchKernelGGL((k_csr_spmv_part<true, false, false, false>), dim3(per_part * A.P), dim3(kBlock), A.range_slots * sizeof(double), ds->stream,
                               pa, A.rows, part_ptrs(ds, A), x);
        else if (A.unit)   // squares, if any, are in the scaled vector
            hipLaunchKernelGGL((k_csr_spmv_part<false, false, false, true>), dim3(per_part * A.P), dim3(kBlock), 0, ds->stream, pa, A.rows,
                               part_ptrs(ds, A), x);
        else if (square)
            hipLaunchKernelGGL((k_csr_spmv_part<false, false, true, false>), dim3(per_part * A.P), dim3(kBlock), 0, ds->stream, pa, A.rows,
                               part_ptrs(ds, A), x);
        else
            hipLaunchKernelGGL((k_csr_spmv_part<false, false, false, false>), dim3(per_part * A.P), dim3(kBlock), 0, ds->stream, pa, A.rows,
                               part_ptrs(ds, A), x);
        TRON_HIP(hipGetLastError());
    }
    TRON_TRY(launch_fixup<EPI_PLAIN>(ds, A, ds->row_partials, nullptr, 0.0));
    return TRON_OK;
}

int spmv_loss(tron_dataset *ds, const CsrPlan &A, int slot, int loss, const double *x, double *zwork, double *zhat, double *D,
              const double *post, int first)
{
    if (single_sums(A) && !post) {
        const EpiArgs E{zhat, ds->y, 0.0, false, D, ds->partials, finish_for(ds, first, A.nblocks)};
        return loss == TRON_LOSS_LR ? launch_single<EPI_LR>(ds, A, slot, x, E) : launch_single<EPI_SVM>(ds, A, slot, x, E);
    }
    if (A.plain) {
        if (post) { set_error("internal: post-scaling on an unpartitioned plan"); return TRON_EINVAL; }
        TRON_TRY(launch_plain<EPI_PLAIN>(ds, A, slot, x, zwork, nullptr, 0.0));
        return loss_terms(ds, loss, zwork, zhat, D, first);
    }
    TRON_TRY(launch_partials(ds, A, slot, x));
    ProfScope ps(ds, SLOT_SPMV_COMBINE);
    const int g = vec_grid(A.rows);
    const Finish fin = finish_for(ds, first, g);
    if (loss == TRON_LOSS_LR)
        hipLaunchKernelGGL(k_combine_loss<TRON_LOSS_LR>, dim3(g), dim3(kBlock), 0, ds->stream, A.rows, partial_ref(ds, A), ds->y, zhat, D, ds->partials, post, fin);
    else
        hipLaunchKernelGGL(k_combine_loss<TRON_LOSS_L2SVM>, dim3(g), dim3(kBlock), 0, ds->stream, A.rows, partial_ref(ds, A), ds->y, zhat, D, ds->partials, post, fin);
    TRON_HIP(hipGetLastError());
    return g;
}

int spmv_scale(tron_dataset *ds, const CsrPlan &A, int slot, const double *x, const double *scale, double *out, const double *post)
{
    if (A.direct && !post) {
        const int g = launch_single<EPI_SCALE>(ds, A, slot, x, EpiArgs{out, scale, 0.0, false, nullptr, nullptr, no_finish(ds)});
        return g < 0 ? g : TRON_OK;
    }
    if (A.plain) {
        if (post) { set_error("internal: post-scaling on an unpartitioned plan"); return TRON_EINVAL; }
        return launch_plain<EPI_SCALE>(ds, A, slot, x, out, scale, 0.0);
    }
    TRON_TRY(launch_partials(ds, A, slot, x));
    ProfScope ps(ds, SLOT_SPMV_COMBINE);
    hipLaunchKernelGGL(k_combine_scale, dim3(vec_grid(A.rows)), dim3(kBlock), 0, ds->stream, A.rows, partial_ref(ds, A), scale, out, post);
    TRON_HIP(hipGetLastError());
    return TRON_OK;
}

// xs = x .* scale  (or x .* scale^2)
__global__ __launch_bounds__(kBlock) void k_prescale(int64_t m, const double *__restrict__ x, const double *__restrict__ scale,
                                                     int square, double *__restrict__ xs)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m; i += (int64_t)gridDim.x * kBlock) {
        const double r = scale[i];
        xs[i] = x[i] * (square ? r * r : r);
    }
}

int spmv_axpy(tron_dataset *ds, const CsrPlan &A, int slot, const double *x, const double *add, double alpha, bool dot_self,
              double *out, bool square, bool x_prescaled, int first)
{
    if (square && A.hot_ids) { set_error("internal: squared product on a layout with LDS tables"); return TRON_EINVAL; }
    if (A.unit && A.col_scale && !x_prescaled) {
        // the plan gathers from x .* col_scale (the entries themselves carry no values)
        ProfScope ps(ds, SLOT_SPMV_GATHER);
        hipLaunchKernelGGL(k_prescale, dim3(vec_grid(A.cols)), dim3(kBlock), 0, ds->stream, A.cols, x, A.col_scale, square ? 1 : 0, A.xs);
        TRON_HIP(hipGetLastError());
        x = A.xs;
    } else if (x_prescaled && !(A.unit && A.col_scale)) {
        set_error("internal: pre-scaled vector for a plan without column scale");
        return TRON_EINVAL;
    }
    if (single_sums(A)) {
        const int g = launch_single<EPI_AXPY>(ds, A, slot, x, EpiArgs{out, add, alpha, dot_self, nullptr, add ? ds->partials : nullptr, finish_for(ds, add ? first : -1, A.nblocks)}, square);
        return (g < 0 || add) ? g : 0;
    }
    if (A.plain) {
        TRON_TRY(launch_plain<EPI_AXPY>(ds, A, slot, x, out, add, alpha, square));
        if (!add) return 0;
        return dot_partials(ds, A.rows, out, dot_self ? out : add, nullptr, nullptr, nullptr, nullptr, first);
    }
    HotRef hot{nullptr, nullptr};
    if (A.hot.ntiles_total > 0) {
        TRON_TRY(launch_hot_tiles(ds, A, x, square));
        hot.slot_of_row = A.hot.slot_of_row;
        hot.sums = A.hot.sums;
    }
    TRON_TRY(launch_partials(ds, A, slot, x, square));
    ProfScope ps(ds, SLOT_SPMV_COMBINE);
    const int g = vec_grid(A.rows);
    const Finish fin = finish_for(ds, add ? first : -1, g);
    if (dot_self)
        hipLaunchKernelGGL(k_combine_axpy<true>, dim3(g), dim3(kBlock), 0, ds->stream, A.rows, partial_ref(ds, A), add, alpha, out, ds->partials, hot, fin);
    else
        hipLaunchKernelGGL(k_combine_axpy<false>, dim3(g), dim3(kBlock), 0, ds->stream, A.rows, partial_ref(ds, A), add, alpha, out, ds->partials, hot, fin);
    TRON_HIP(hipGetLastError());
    return g;
}

// ------------------------------------------------------------------ byte accounting (see PlanBytes)
PlanBytes plan_bytes(const CsrPlan &A)
{
    PlanBytes b{0, 0, 0, 0, 0, 0};
    const int64_t vbytes = A.unit ? 0 : 8;   // value stream per stored entry
    if (A.plain) {
        // plain CSR in chunks: columns and values once, row offsets, the gathered vector and the result once each
        b.ranges = A.part_nnz[0] * (4 + 8) + 8 * (A.rows + 1) + 4 * ((int64_t)A.nblocks + 1) + 8 * A.cols + 8 * A.rows;
        return b;
    }
    const int64_t per_chunk = kBlock /* flag bits */ + (int64_t)sizeof(int4) /* table entry */ + 8 /* carry */;
    int64_t nseg_head = 0;
    if (A.hot_ids) {
        const int64_t nh = (int64_t)A.P * kHotSlots + A.head_slots;
        b.gather = nh * (4 + 8 + 8);
    }
    if (A.sell.on) {
        b.head = A.sell.ngroups * kWave * 16 + 8 * ((int64_t)A.sell.nwaves + 1) + 8 * (int64_t)kSellSlots + 8 * A.sell.nrows_with_entries;
    } else if (A.head >= 0) {
        const int h = A.head;
        nseg_head = A.nseg_total - A.part_seg0[h];
        b.head = (int64_t)A.part_nchunks[h] * (kChunk * (2 + vbytes) + per_chunk) + 8 * (int64_t)kHotSlots + 8 * nseg_head;
    }
    int64_t range_chunks = 0;
    for (int x = 0; x < A.P; ++x) range_chunks += A.part_nchunks[x];
    const int64_t nseg_ranges = A.nseg_total - nseg_head;
    b.ranges = range_chunks * (kChunk * (4 + vbytes) + per_chunk) + 8 * nseg_ranges + 8 * A.cold_cols +
               (A.hot_ids ? 8 * (int64_t)A.P * A.range_slots : 0);
    if (A.hot.ntiles_total > 0) {
        const HotTiles &H = A.hot;
        const HotWindows &Q = H.win;
        const int64_t acc = Q.on ? 8 * Q.npieces : 8 * (int64_t)kTileSlices * H.blocks_per_slice * kTileSlots;
        if (Q.on) b.tiles = Q.ngroups * kWave * 16 + 8 * (int64_t)kSellWaves * Q.nblocks + 8 * (int64_t)Q.width * Q.nblocks + acc;
        else b.tiles = H.ntiles_total * (kChunk * (2 + vbytes) + kBlock + (int64_t)sizeof(int4)) + 2 * H.nseg_padded + 8 * H.span_total + acc;
        b.tile_reduce = Q.on ? acc + 2 * (int64_t)Q.nwin * Q.nslots + 8 * (int64_t)H.nhot : acc + 8 * (int64_t)kTileSlices * kTileSlots;
    }
    if (A.direct) {   // row ranges and segment numbers, addend and result, no partial sums
        b.ranges += 4 * A.rows + 16 * A.rows - 8 * nseg_ranges;
        return b;
    }
    // combine: every partial sum once, the row mask, the group table, the result; plus what the plan's extras need per row
    b.combine = 8 * A.nseg_total + 2 * A.rows + (int64_t)sizeof(GroupBase) * A.ngroups + 8 * A.rows;
    if (A.sell.on) b.combine += (8 + 4) * A.rows;                        // sorted sums through the position array
    if (A.hot.ntiles_total > 0) b.combine += 4 * A.rows + 8 * (int64_t)A.hot.nhot;   // slot of each row, sums of the hot rows
    if (A.row_scale) b.combine += 8 * A.rows;
    return b;
}

}  // namespace tron
