// Dense row-major kernels: one pass over X computes both products of Table 1 of the paper,
//   Hessian-vector:  X^T ( D (X v) )        (written there as 2C X_I^T (X_I v) for the L2-SVM; the
//                                            active set enters through D_ii in {0, 2})
//   function/gradient:  z = X w, the per-instance loss, zhat and D, and X^T zhat
// so each element of X is read from HBM exactly once per call.
//
// Layout of the work inside a wavefront (64 lanes): a row is covered by L consecutive lanes, each
// holding E of its columns (E*L >= d; see Tile); one "step" covers 64/L rows and a wave tile of
// U steps covers RT = U*64/L consecutive rows.  For d = 24: E = 6, L = 4, U = 4 -- 64 rows = 12 KiB per
// tile, each lane issuing three 16-byte loads per step, twelve per tile, all in flight together.
//   1. partial dot products x.v per lane, summed over the L lanes of the row and folded on the way, so that a
//      row's total ends up in the lanes that own the row;
//   2. the per-row scalar work (sigmoid / log1p for the logistic loss, D scaling) runs in the owners, and D, y
//      are read / written as one coalesced access;
//   3. the per-row coefficient goes back to the row's lanes (moves inside a quad of lanes) and is accumulated into E
//      private column accumulators, which are reduced over the wavefront / workgroup once, at the end.
// Every workgroup leaves its column sums at `partials[block * d ...]`.  For d <= 32 the workgroup that finishes last adds
// them in a fixed order and forms the outputs (dense_finish); the separate launch this replaces took 9.7 us for 2048
// workgroups of 24 columns.  Wider matrices take a launch of k_dense_columns, one workgroup per 16 columns.  Nothing is added
// in an order that depends on timing.
#include <algorithm>
#include <atomic>
#include <cmath>

#include "dense_tile.h"
#include "device_driver.h"
#include "grid_sync.h"

namespace tron {

namespace {

// What the second stage of a pass forms from the per-workgroup column sums:
//   out = add + C * sums (add == null: add 1);  scal null: no scalars;
//   fun_grad: scal[0] = sum of the losses, [1] = add.add (add = w), [2] = out.out, [3] = rows with D != 0;
//   otherwise: scal[0] = scal_copy[0] = out.dotw (the CG step kernel continues from the copy).
struct DenseFinish {
    unsigned *ticket;      // counter of finished workgroups (zero between kernels); d <= 32: null = the pass leaves its sums alone
    const double *add;
    double C;
    double *out;           // may be null
    const double *dotw;    // null: out itself
    double *scal, *scal_copy;
    bool fun_grad;
    HostFlag flag;         // with scal
};

// d <= 32 (at most four lanes per row): the last workgroup completes the sums
constexpr bool dense_finishes(int L) { return L <= 4; }
constexpr int kFinishMaxD = 32;
// Eight wavefronts per CU: with twelve loads of 16 bytes per lane in flight they keep HBM busy, and every workgroup more costs its
// ticket (10 ns, one after the other) and its sums.  More only for narrow rows (tiles_at_once, dense_fun_grad_grid) and for few
// active ones (kFewBelow).  1M x 24, a Hessian-vector call with 256 / 512 / 1024 / 2048 workgroups: 43 / 44 / 52 / 64 us; 20M x 24: 629 / 640 / 652 / 663 us.  Twelve wavefronts: 44 and 633 us.
constexpr int dense_block(int L) { return dense_finishes(L) ? 512 : kBlock; }
constexpr int kFinishGrid = 256, kWideGrid = 512, kFewGrid = 512;
// doubles of LDS: the column sums of the wavefronts, then one per thread for the workgroup that finishes last
constexpr int dense_lds(int E, int L) { return dense_block(L) / kWave * E * L > dense_block(L) ? dense_block(L) / kWave * E * L : dense_block(L); }
constexpr int kColumnsBlock = 1024, kColumnsPer = 16;

__device__ __forceinline__ void store_dense_scalars(const DenseFinish &fin, double loss, double ww, double cp, double active)
{
    if (fin.fun_grad) {
        store_host(fin.scal, loss);
        store_host(fin.scal + 1, ww);
        store_host(fin.scal + 2, cp);
        store_host(fin.scal + 3, active);
    } else {
        store_host(fin.scal, cp);
        fin.scal_copy[0] = cp;
    }
}

// One workgroup adds the rows of partial sums of `grid` workgroups, d <= 32: thread t the elements t, t + T, ... of the
// d x grid array, T a multiple of d, so all of them belong to column t % d; then over the threads of a column in LDS (col_sum:
// a double per thread; its earlier contents have been read by wavefront 0 only).  True in wavefront 0: lane c < d then has
// column c's sum, every lane the loss sum and the number of active rows (zero without loss_partials; the latter
// also without active_partials).
template <int kWaves>
__device__ __forceinline__ bool dense_add_rows(double *col_sum, int grid, int d, const double *partials, const double *loss_partials,
                                               const double *active_partials, double &col, double &loss, double &active)
{
    constexpr int kThreads = kWaves * kWave, kAtOnce = 8;
    __shared__ double red[2][kWaves];
    const int t = threadIdx.x, lane = t & (kWave - 1), wv = t / kWave;
    const int groups = kThreads / d, T = groups * d, total = d * grid;
    double s = 0.0;
    if (t < T)
        for (int i0 = t; i0 < total; i0 += kAtOnce * T) {
            double v[kAtOnce];
#pragma unroll
            for (int k = 0; k < kAtOnce; ++k) v[k] = (i0 + k * T < total) ? load_shared(partials + i0 + k * T) : 0.0;
#pragma unroll
            for (int k = 0; k < kAtOnce; ++k) s += v[k];
        }
    col_sum[t] = s;
    double a = 0.0, e = 0.0;
    if (loss_partials) {
        for (int b = t; b < grid; b += kThreads) {
            a += load_shared(loss_partials + b);
            if (active_partials) e += load_shared(active_partials + b);
        }
        a = wave_sum(a);
        e = wave_sum(e);
    }
    if (lane == 0) {
        red[0][wv] = a;
        red[1][wv] = e;
    }
    __syncthreads();
    if (wv != 0) return false;
    // m lanes share a column's groups, m the largest power of two with d m <= 64: eight to sixteen additions one after the
    // other whatever d is.  With one lane per column they were 512 / d: a Hessian-vector call over 100,000 rows
    // took 11.9 us at d = 1 (6.9 now), 9.0 at d = 4 (7.9), 9.4 at d = 24 (9.3).
    const int m = kWave >> (d > 1 ? 32 - __clz(d - 1) : 0), c = lane / m;
    col = loss = active = 0.0;
    if (c < d)
        for (int k0 = lane % m; k0 < groups; k0 += kAtOnce * m) {
            double v[kAtOnce];
#pragma unroll
            for (int k = 0; k < kAtOnce; ++k) v[k] = (k0 + k * m < groups) ? col_sum[(k0 + k * m) * d + c] : 0.0;
#pragma unroll
            for (int k = 0; k < kAtOnce; ++k) col += v[k];
        }
    col = __shfl(group_sum(col, m), lane * m, kWave);
    if (lane >= d) col = 0.0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        loss += red[0][k];
        active += red[1][k];
    }
    return true;
}

// Every thread of every workgroup calls it; wavefront 0 has written the workgroup's column sums (and its two other sums) last.
// The workgroup that draws the last ticket adds the rows; the caller clears the counter.
template <int kWaves>
__device__ __forceinline__ bool dense_last_sums(double *col_sum, unsigned *ticket, int d, const double *partials, const double *loss_partials,
                                                const double *active_partials, double &col, double &loss, double &active)
{
    return last_workgroup(ticket) && dense_add_rows<kWaves>(col_sum, (int)gridDim.x, d, partials, loss_partials, active_partials, col, loss, active);
}

// what wavefront 0 forms from the sums: the outputs and the scalars
__device__ __forceinline__ void dense_outputs(const DenseFinish &fin, int d, double sum, double loss, double active)
{
    const int lane = threadIdx.x;
    double cp = 0.0, ww = 0.0;
    if (lane < d) {
        const double add = fin.add ? fin.add[lane] : 1.0;
        const double o = fma(fin.C, sum, add);
        cp = o * (fin.dotw ? fin.dotw[lane] : o);
        ww = add * add;
        if (fin.out) store_shared(fin.out + lane, o);
    }
    cp = wave_sum(cp);
    ww = wave_sum(ww);
    if (lane == 0 && fin.scal) store_dense_scalars(fin, loss, ww, cp, active);
    post_flag(fin.flag);
}

template <int kWaves>
__device__ __forceinline__ void dense_finish(double *lds, const DenseFinish &fin, int d, const double *partials, const double *loss_partials,
                                             const double *active_partials)
{
    double sum, loss, active;
    if (!dense_last_sums<kWaves>(lds, fin.ticket, d, partials, loss_partials, active_partials, sum, loss, active)) return;
    dense_outputs(fin, d, sum, loss, active);
    if (threadIdx.x == 0) *fin.ticket = 0u;
}

// The same as a launch of its own behind a pass without a counter (tron_hv_static): the same sums in the same order.
constexpr int kFinishBlock = dense_block(1);
__global__ __launch_bounds__(kFinishBlock) void k_dense_finish(int d, int grid, const double *__restrict__ partials, DenseFinish fin)
{
    __shared__ double lds[kFinishBlock];
    double sum, loss, active;
    if (dense_add_rows<kFinishBlock / kWave>(lds, grid, d, partials, nullptr, nullptr, sum, loss, active)) dense_outputs(fin, d, sum, loss, active);
}

// Tiles whose loads a wavefront of the Hessian-vector pass issues together: a tile of narrow rows is only 512 d bytes, and eight
// wavefronts per CU with one such tile each do not keep HBM busy.  Up to d = 4 those in flight on a CU still fit its 32 KB L1,
// which serves a lane's loads of the same line (d <= 8: a lane holds a whole row); two tiles at d = 5 gain nothing, and at d = 4
// only where D is one bit a row (mask).  20M rows, one tile / several, L2-SVM: d = 1 57 / 30 us, 2 92 / 51, 3 108 / 81,
// 4 117 / 104; logistic: 94 / 55, 103 / 81, 116 / 105, 126 / 132.
constexpr int tiles_at_once(int E, int L, bool mask) { return L > 1 ? 1 : E == 1 ? 8 : E == 2 ? 4 : E == 3 || (E == 4 && mask) ? 2 : 1; }

// The tiles of a wavefront: first, first + step, ... below last.  A contiguous range, or every tile whose number leaves the
// wavefront's as remainder.
struct TileWalk {
    int64_t first, last, step;
    __device__ __forceinline__ TileWalk(int64_t ntiles, int waves, bool contiguous)
    {
        const int64_t nwaves = (int64_t)gridDim.x * waves, id = (int64_t)blockIdx.x * waves + threadIdx.x / kWave;
        const int64_t per = (ntiles + nwaves - 1) / nwaves;
        first = contiguous ? id * per : id;
        last = contiguous && first + per < ntiles ? first + per : ntiles;
        step = contiguous ? 1 : nwaves;
    }
};

// D has arrived when the call that computes it returns, which is some microseconds before the kernel ends that gives the word for
// it: a captured tron_hv_static may be replayed on another stream from then on.  (Rows of more than four lanes: the word comes from the
// kernel after the pass.  With these stores 200,003 x 257 would take 340 us instead of 336.)
template <int L, typename T>
__device__ __forceinline__ void store_D(T *p, T v)
{
    if constexpr (dense_finishes(L)) store_shared(p, v);
    else *p = v;
}

// ------------------------------------------------------------------ Hessian-vector pass
// MASK: D is the active set of the L2-SVM (D_ii = 2 on it, else 0) instead of an fp64 value per row: one bit per row,
// a 64-bit word per wave tile, when a tile has 64 rows (d <= 32); one byte per row otherwise.
// DIAG: column sums of D_i x_ij^2 instead (the diagonal of X^T D X; v is not read).
// SKIP (with the bit words only): rows outside the active set are not read.  Chosen by the host when a noticeable
// part of the rows is inactive; with (almost) every row active the plain loop is about 1% faster.
// STREAM: X comes through LDS (TileStream; every row is read).
// SOLVE: the pass is one of several in a launch.  All of them then deal the tiles out alike, so that a wavefront reads the D that
// it wrote itself.
// lds: E * L doubles per wavefront
template <int E, int L, int U, bool VEC, bool MASK, bool DIAG, bool SKIP, bool STREAM, bool SOLVE = false>
__device__ __forceinline__ void hv_pass(double *lds, int64_t n, int64_t d, const double *__restrict__ X, const void *__restrict__ Dv,
                                        const double *__restrict__ v, double *__restrict__ partials, double *stream_lds)
{
    constexpr int kWaves = dense_block(L) / kWave;
    const double *D = static_cast<const double *>(Dv);
    const uint8_t *Dm = static_cast<const uint8_t *>(Dv);
    using T = Tile<E, L, U, VEC>;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int q = lane % L, own = T::own_row(lane);
    double vreg[E], acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        vreg[e] = (!DIAG && T::col(q, e) < d) ? v[T::col(q, e)] : 0.0;
        acc[e] = 0.0;
    }
    const int64_t ntiles = (n + T::RT - 1) / T::RT;
    // With the active set as one 64-bit word per tile (bit i = row row0 + i is active; rows past n are never set)
    // the rows outside it are not read: the pass moves 8 |I| d bytes, the saving the paper gets from a compacted
    // copy X_I (Section 5) without the copy.  The word of the next tile is fetched one iteration ahead.
    constexpr bool kBits = MASK && T::RT == kWave;
    const uint64_t *Dbits = static_cast<const uint64_t *>(Dv);
    constexpr int G = tiles_at_once(E, L, MASK);
    const TileWalk walk(ntiles, kWaves, SOLVE && kBits);
    const int64_t tile0 = walk.first, last = walk.last, nwaves = walk.step;
    // the products of a tile whose rows' D are in Drow
    auto add_tile = [&](const double (&x)[U][E], double Drow) {
        double c[U];
        if (DIAG) {
            T::from_row_owner(Drow, c);
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = fma(c[u] * x[u][e], x[u][e], acc[e]);
            }
        } else {
            T::from_row_owner(Drow * T::row_sum(x, vreg, lane), c);   // a1 = D (X v)
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = fma(c[u], x[u][e], acc[e]);
            }
        }
    };
    if constexpr (STREAM) {
        static_assert(!SKIP, "");
        TileStream<E, L, U, VEC> stream(stream_lds, d);
        // D of a tile travels with its rows
        uint64_t bits = 0;
        double Drow = 0.0;
        auto ask = [&](int64_t t) {
            stream.ask(X, n, d, t, t < last);
            if (kBits) bits = t < last ? Dbits[t] : 0;
            else if (t < last && t * T::RT + own < n) Drow = MASK ? (Dm[t * T::RT + own] ? 2.0 : 0.0) : D[t * T::RT + own];
            else Drow = 0.0;
        };
        ask(tile0);
        for (int64_t tile = tile0; tile < last; tile += nwaves) {
            double x[U][E];
            stream.take(X, n, d, tile, lane, x);
            const double mine = kBits ? (((bits >> own) & 1u) ? 2.0 : 0.0) : Drow;
            ask(tile + nwaves);
            add_tile(x, mine);
        }
    } else {
        uint64_t bits_next[G];
#pragma unroll
        for (int g = 0; g < G; ++g) bits_next[g] = (kBits && SKIP && tile0 + g * nwaves < last) ? Dbits[tile0 + g * nwaves] : 0;
        for (int64_t tile = tile0; tile < last; tile += G * nwaves) {
            double x[G][U][E], Drow[G];
            uint64_t bits[G], any = 0;
            if (kBits && SKIP) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int64_t ahead = tile + (G + g) * nwaves;
                    bits[g] = bits_next[g];
                    any |= bits[g];
                    bits_next[g] = (ahead < last) ? Dbits[ahead] : 0;
                }
                if (any == 0) continue;   // no active row in the tiles
            }
            // tiles past the last one: every row is past n
#pragma unroll
            for (int g = 0; g < G; ++g) T::load(X, n, d, ((SOLVE && tile + g * nwaves >= last) ? ntiles : tile + g * nwaves) * T::RT, lane, x[g], (kBits && SKIP) ? bits[g] : ~0ull);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int64_t t = tile + g * nwaves, row = t * T::RT + own;
                if (kBits && !SKIP) bits[g] = (t < last) ? Dbits[t] : 0;
                Drow[g] = 0.0;
                if (kBits) {
                    Drow[g] = ((bits[g] >> own) & 1u) ? 2.0 : 0.0;
                } else if (row < n) {
                    Drow[g] = MASK ? (Dm[row] ? 2.0 : 0.0) : D[row];
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) add_tile(x[g], Drow[g]);
        }
    }
    T::flush(acc, d, lane, wv, kWaves, lds, partials + (int64_t)blockIdx.x * d, 1);
}

template <int E, int L, int U, bool VEC, bool MASK, bool DIAG, bool SKIP, bool STREAM>
__global__ __launch_bounds__(dense_block(L)) void k_dense_hv(int64_t n, int64_t d, const double *__restrict__ X,
                                                                const void *__restrict__ Dv, const double *__restrict__ v,
                                                                double *__restrict__ partials, DenseFinish fin)
{
    constexpr int kWaves = dense_block(L) / kWave;
    __shared__ double lds[dense_lds(E, L)];
    // the counter of k_dense_columns starts at zero whatever an earlier call left in it
    if constexpr (!dense_finishes(L)) { if (blockIdx.x == 0 && threadIdx.x == 0) *fin.ticket = 0u; }
    extern __shared__ __align__(16) double stream_lds[];
    hv_pass<E, L, U, VEC, MASK, DIAG, SKIP, STREAM>(lds, n, d, X, Dv, v, partials, stream_lds);
    if constexpr (dense_finishes(L)) { if (fin.ticket) dense_finish<kWaves>(lds, fin, (int)d, partials, nullptr, nullptr); }
}

// ------------------------------------------------------------------ function / gradient pass
// lds as in hv_pass, lds_red: two rows of one double per wavefront
template <int E, int L, int U, bool VEC, int LOSS, bool STREAM>
__device__ __forceinline__ void fun_grad_pass(double *lds, double (*lds_red)[dense_block(L) / kWave], int64_t n, int64_t d,
                                              const double *__restrict__ X, const int8_t *__restrict__ y, const double *__restrict__ w,
                                              void *__restrict__ Dv, double *__restrict__ partials,
                                              double *__restrict__ loss_partials, double *__restrict__ active_partials, double *stream_lds)
{
    using T = Tile<E, L, U, VEC>;
    constexpr int kWaves = dense_block(L) / kWave;
    double *Dout = static_cast<double *>(Dv);       // logistic loss: fp64 D
    uint8_t *Dmask = static_cast<uint8_t *>(Dv);    // L2-SVM: active-set mask
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int q = lane % L, own = T::own_row(lane);
    double wreg[E], acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        wreg[e] = (T::col(q, e) < d) ? w[T::col(q, e)] : 0.0;
        acc[e] = 0.0;
    }
    LossSum<LOSS> losses;
    double active_acc = 0.0;   // number of rows with D != 0
    // Active set of the L2-SVM when a tile has 64 rows: one 64-bit word per tile.  A wavefront then walks a
    // contiguous range of tiles, lane i keeps the word of its i-th, 64+i-th, ... tile, and every 64 tiles the words
    // go out as one 512-byte store: small stores between the reads cost far more than their bytes.
    constexpr bool kBits = (LOSS == TRON_LOSS_L2SVM) && (T::RT == kWave);
    uint64_t *Dbits = static_cast<uint64_t *>(Dv);
    uint64_t held_bits = 0;
    int64_t held_tile = -1;
    const int64_t ntiles = (n + T::RT - 1) / T::RT;
    const TileWalk walk(ntiles, kWaves, kBits);
    const int64_t first = walk.first, last = walk.last, step = walk.step;
    int it = 0;
    TileStream<E, L, U, VEC> stream(STREAM ? stream_lds : nullptr, d);
    int8_t label = 1;   // of the lane's row of a tile that comes through LDS: travels with it
    // logistic D of the tile before: stored before the next tile is asked for, as the wait for that one is a wait for the store, too
    double D_held = 0.0;
    int64_t D_row = -1;
    auto ask = [&](int64_t t) {
        if (!STREAM) return;
        label = t < last && t * T::RT + own < n ? y[t * T::RT + own] : 1;
        stream.ask(X, n, d, t, t < last);
    };
    ask(first);
    for (int64_t tile = first; tile < last; tile += step, ++it) {
        const int64_t row0 = tile * T::RT;
        double x[U][E], c[U];
        if (STREAM) stream.take(X, n, d, tile, lane, x);
        else T::load(X, n, d, row0, lane, x);
        const bool in = row0 + own < n, mine = in && T::first_owner(lane);
        if (STREAM && !kBits && D_row >= 0) store_D<L>(Dout + D_row, D_held);
        const double yrow = STREAM ? (double)label : in ? (double)y[row0 + own] : 1.0;
        ask(tile + step);
        const double z = T::row_sum(x, wreg, lane);           // z = X w
        LossTerm alpha;
        double zhat, Di;
        loss_terms_dev<LOSS>(z, yrow, alpha, zhat, Di);
        if (mine) {
            losses.add(alpha);
            active_acc += (Di != 0.0) ? 1.0 : 0.0;
        }
        if (!in) {
            Di = 0.0;
            zhat = 0.0;
        }
        if (kBits) {
            const uint64_t bits = T::ballot_rows(Di != 0.0, lane);
            if (lane == (it & (kWave - 1))) { held_bits = bits; held_tile = tile; }
            if ((it & (kWave - 1)) == kWave - 1) {
                store_shared(Dbits + held_tile, held_bits);   // every lane holds one: 64 consecutive words
                held_tile = -1;
            }
        } else if (STREAM) {
            D_held = Di;
            D_row = mine ? row0 + own : -1;
        } else if (mine) {
            if (LOSS == TRON_LOSS_L2SVM) store_D<L>(Dmask + row0 + own, (uint8_t)(Di != 0.0 ? 1 : 0));
            else store_D<L>(Dout + row0 + own, Di);
        }
        if ((it & (LossSum<LOSS>::kAdds - 1)) == LossSum<LOSS>::kAdds - 1) losses.scale();
        T::from_row_owner(zhat, c);
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = fma(c[u], x[u][e], acc[e]);
        }
    }
    if (kBits && held_tile >= 0) store_shared(Dbits + held_tile, held_bits);
    if (STREAM && !kBits && D_row >= 0) store_D<L>(Dout + D_row, D_held);
    if (dense_finishes(L)) stores_arrived();   // before the workgroup's ticket: the host goes on when the last one has been drawn
    const double loss_acc = wave_sum(losses.value());
    active_acc = wave_sum(active_acc);
    if (lane == 0) {
        lds_red[0][wv] = loss_acc;
        lds_red[1][wv] = active_acc;
    }
    T::flush(acc, d, lane, wv, kWaves, lds, partials + (int64_t)blockIdx.x * d, 1);
    if (threadIdx.x < (active_partials ? 2 : 1)) {   // (a solve does not count them)
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) t += lds_red[threadIdx.x][k];
        store_shared((threadIdx.x ? active_partials : loss_partials) + blockIdx.x, t);
    }
}

template <int E, int L, int U, bool VEC, int LOSS, bool STREAM>
__global__ __launch_bounds__(dense_block(L)) void k_dense_fun_grad(int64_t n, int64_t d, const double *__restrict__ X,
                                                                      const int8_t *__restrict__ y, const double *__restrict__ w,
                                                                      void *__restrict__ Dv, double *__restrict__ partials,
                                                                      double *__restrict__ loss_partials, double *__restrict__ active_partials,
                                                                      DenseFinish fin)
{
    constexpr int kWaves = dense_block(L) / kWave;
    __shared__ double lds[dense_lds(E, L)];
    __shared__ double lds_red[2][kWaves];
    extern __shared__ __align__(16) double stream_lds[];
    fun_grad_pass<E, L, U, VEC, LOSS, STREAM>(lds, lds_red, n, d, X, y, w, Dv, partials, loss_partials, active_partials, stream_lds);
    if constexpr (dense_finishes(L)) dense_finish<kWaves>(lds, fin, (int)d, partials, loss_partials, active_partials);
}

// ------------------------------------------------------------------ a solve driven from the device
// Passes that serve the problem's pending request -- function / gradient at a trial point or a Hessian-vector product -- each followed
// by the step of Algorithm 1 or of the CG iteration that was waiting for it.  d <= 32, tiles of 64 rows.
// stamp == 0: the whole solve in one launch of workgroups that are all resident.  Every workgroup keeps the problem's state in LDS,
// adds all partial sums and takes the step itself (in the same order, so all hold the same bits): between two passes lies one
// barrier over the grid.  Only the first workgroup reports.  A round of 20,000 x 24 takes 7.6 us (the pass with its tile in registers 2.3, the
// barrier 2, the sums 1.5, the step 1.5), as a launch of its own 10 and the gaps; whole solves 72 us with a launch per round, 50 in
// one; 1M x 24 215 and 175 (144 to 188 from box to box); 5M x 18 logistic 748 and 706.
// ROWS_KEPT: no wavefront has more than one tile (stamp == 0 only).
// stamp > 0: round `stamp` of a solve with a launch per round (grids of more workgroups than CUs, solves of other threads that
// leave no room, see ResidentShare, or a part of the GPU held otherwise): the workgroup that finishes last adds the sums and takes the step, the state lies in device memory.  The
// same sums in the same order, the same results.
struct SolveArgs {
    const double *X;
    const int8_t *y;
    void *D[2];
    double *partials, *loss_partials;
    int64_t round_stride;   // doubles between the partial sums of even and odd rounds (a workgroup may be one round ahead)
    unsigned *ticket;
    GridSync sync;
    BatchCtl *ctl;
    ProbState *st;
    const double *w0;       // stamp == 0: the starting point
    double C;
    tron_trace_rec *trace;
    BatchHost *host;
};

// Either pass of a solve over so few rows that a wavefront has one tile at most: the tile, its labels and the two D buffers' entries
// of the lane's row stay in registers for the whole solve (D goes to memory as well, for the calls after the solve).  The same
// operations in the same order as fun_grad_pass and hv_pass.  20,000 x 24: 1.2 us a pass instead of 3.
template <int E, int L, int U, bool VEC, int LOSS>
struct OneTile {
    using T = Tile<E, L, U, VEC>;
    static constexpr int kWaves = dense_block(L) / kWave;
    static constexpr bool svm = LOSS == TRON_LOSS_L2SVM;
    double x[U][E], y, Dreg[2];
    bool in;

    __device__ __forceinline__ void load(int64_t n, int64_t d, const double *__restrict__ X, const int8_t *__restrict__ y8)
    {
        const int lane = threadIdx.x & (kWave - 1);
        const int64_t row0 = ((int64_t)blockIdx.x * kWaves + threadIdx.x / kWave) * T::RT, row = row0 + T::own_row(lane);
        in = row < n;
        T::load(X, n, d, row0, lane, x);
        y = in ? (double)y8[row] : 1.0;
        Dreg[0] = Dreg[1] = 0.0;
    }

    __device__ __forceinline__ void pass(double *lds, double (*lds_red)[kWaves], const bool fg, const int slot, int64_t d, const double *vec, void *Dv,
                                         double *__restrict__ partials, double *__restrict__ loss_partials)
    {
        const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave, q = lane % L;
        const int64_t tile = (int64_t)blockIdx.x * kWaves + wv;
        double vreg[E], acc[E], c[U], coef;
#pragma unroll
        for (int e = 0; e < E; ++e) vreg[e] = (T::col(q, e) < d) ? vec[T::col(q, e)] : 0.0;
        const double z = T::row_sum(x, vreg, lane);
        LossSum<LOSS> losses;
        if (fg) {   // uniform
            LossTerm alpha;
            double zhat, Di;
            loss_terms_dev<LOSS>(z, y, alpha, zhat, Di);
            if (in && T::first_owner(lane)) losses.add(alpha);
            Di = in ? Di : 0.0;
            coef = in ? zhat : 0.0;
            if (svm) {
                const uint64_t word = T::ballot_rows(Di != 0.0, lane);
                if (lane == 0 && __ballot(in) != 0) store_shared(static_cast<uint64_t *>(Dv) + tile, word);
            } else if (in && T::first_owner(lane)) {
                store_shared(static_cast<double *>(Dv) + tile * T::RT + T::own_row(lane), Di);
            }
            Dreg[0] = slot ? Dreg[0] : Di;
            Dreg[1] = slot ? Di : Dreg[1];
        } else {
            coef = (slot ? Dreg[1] : Dreg[0]) * z;   // a1 = D (X v)
        }
        T::from_row_owner(coef, c);
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = fma(c[u], x[u][e], acc[e]);
        }
        const double loss_acc = fg ? wave_sum(losses.value()) : 0.0;
        if (lane == 0) lds_red[0][wv] = loss_acc;
        T::flush(acc, d, lane, wv, kWaves, lds, partials + (int64_t)blockIdx.x * d, 1);
        if (threadIdx.x == 0) {
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < kWaves; ++k) t += lds_red[0][k];
            store_shared(loss_partials + blockIdx.x, t);
        }
    }
};

// Either pass of an L2-SVM solve over more rows, one tile at a time: fun_grad_pass and hv_pass in one loop, the same operations in the
// same order.  x holds the wavefront's first tile already where `loaded` is set: it was asked for before the wait for the other
// workgroups, which saves 2 us of a pass of 27 (1M x 24).  The logistic loss keeps its two loops: one for both took 730 us a solve of
// 5M x 18 instead of 718.
template <int E, int L, int U, bool VEC, bool STREAM>
__device__ __forceinline__ void svm_solve_pass(double *lds, double (*lds_red)[dense_block(L) / kWave], const bool fg, int64_t n, int64_t d,
                                               const double *__restrict__ X, const int8_t *__restrict__ y, const double *vec, uint64_t *Dbits,
                                               double *__restrict__ partials, double *__restrict__ loss_partials, double (&x)[U][E], const bool loaded,
                                               TileStream<E, L, U, VEC> &stream)
{
    using T = Tile<E, L, U, VEC>;
    constexpr int kWaves = dense_block(L) / kWave;
    static_assert(T::RT == kWave, "one 64-bit word per tile");
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int q = lane % L, own = T::own_row(lane);
    double vreg[E], acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        vreg[e] = (T::col(q, e) < d) ? vec[T::col(q, e)] : 0.0;
        acc[e] = 0.0;
    }
    const int64_t ntiles = (n + T::RT - 1) / T::RT;
    const TileWalk walk(ntiles, kWaves, true);
    LossSum<TRON_LOSS_L2SVM> losses;
    uint64_t held_bits = 0, bnext = (!fg && walk.first < walk.last) ? Dbits[walk.first] : 0;
    int64_t held_tile = -1;
    int it = 0;
    constexpr int kLeastActive = 48;
    // through LDS: the word of the tile after the next one, too, as the next one's says how its rows come
    uint64_t bnext2 = (STREAM && !fg && walk.first + 1 < walk.last) ? Dbits[walk.first + 1] : 0;
    int8_t label = STREAM && fg && walk.first < walk.last && walk.first * T::RT + own < n ? y[walk.first * T::RT + own] : 1;
    auto ask = [&](int64_t t) {
        if (!STREAM) return;
        bnext = bnext2;
        bnext2 = (!fg && t + 1 < walk.last) ? Dbits[t + 1] : 0;
        if (fg) label = t < walk.last && t * T::RT + own < n ? y[t * T::RT + own] : 1;
        stream.ask(X, n, d, t, t < walk.last && (fg || __popcll(bnext) >= kLeastActive));
    };
    for (int64_t tile = walk.first; tile < walk.last; ++tile, ++it) {
        const int64_t row0 = tile * T::RT;
        const uint64_t bits = bnext;   // fetched one step ahead
        const int8_t label_there = label;
        if (!STREAM) bnext = (!fg && tile + 1 < walk.last) ? Dbits[tile + 1] : 0;
        if (STREAM && stream.there) {
            stream.take(X, n, d, tile, lane, x);
            ask(tile + 1);
        } else {
            ask(tile + 1);
            if (!fg && bits == 0) continue;   // no active row in the tile
            if (STREAM || it > 0 || !loaded) T::load(X, n, d, row0, lane, x, fg ? ~0ull : bits);
            if (STREAM) stream.wait_loads();
        }
        double c[U];
        const double z = T::row_sum(x, vreg, lane);
        if (fg) {   // uniform
            const bool in = row0 + own < n;
            LossTerm alpha;
            double zhat, Di;
            loss_terms_dev<TRON_LOSS_L2SVM>(z, STREAM ? (double)label_there : in ? (double)y[row0 + own] : 1.0, alpha, zhat, Di);
            if (in && T::first_owner(lane)) losses.add(alpha);
            const uint64_t word = T::ballot_rows(in && Di != 0.0, lane);
            if (lane == (it & (kWave - 1))) { held_bits = word; held_tile = tile; }
            if ((it & (kWave - 1)) == kWave - 1) {
                store_shared(Dbits + held_tile, held_bits);   // every lane holds one: 64 consecutive words
                held_tile = -1;
            }
            T::from_row_owner(in ? zhat : 0.0, c);
        } else {
            T::from_row_owner((((bits >> own) & 1u) ? 2.0 : 0.0) * z, c);   // a1 = D (X v)
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = fma(c[u], x[u][e], acc[e]);
        }
    }
    if (held_tile >= 0) store_shared(Dbits + held_tile, held_bits);
    stores_arrived();
    const double loss_acc = wave_sum(losses.value());
    if (lane == 0) lds_red[0][wv] = loss_acc;
    T::flush(acc, d, lane, wv, kWaves, lds, partials + (int64_t)blockIdx.x * d, 1);
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) t += lds_red[0][k];
        store_shared(loss_partials + blockIdx.x, t);
    }
}

template <typename T>
__device__ __forceinline__ void copy_words(T *dst, const T *src)
{
    static_assert(sizeof(T) % sizeof(uint64_t) == 0, "");
    for (int i = threadIdx.x; i < (int)(sizeof(T) / sizeof(uint64_t)); i += blockDim.x) reinterpret_cast<uint64_t *>(dst)[i] = reinterpret_cast<const uint64_t *>(src)[i];
}

enum Rows { ROWS_LOADED = 0, ROWS_KEPT, ROWS_STREAMED };   // as a pass needs them, in registers (OneTile), through LDS
template <int E, int L, int U, bool VEC, int LOSS, Rows ROWS>
__global__ __launch_bounds__(dense_block(L)) void k_dense_solve(int64_t n, int64_t d, SolveArgs A, SolveParams P, int64_t stamp)
{
    constexpr int kWaves = dense_block(L) / kWave;
    constexpr bool svm = LOSS == TRON_LOSS_L2SVM, ONE = ROWS == ROWS_KEPT, STREAM = ROWS == ROWS_STREAMED;
    __shared__ double lds[dense_lds(E, L)];
    __shared__ double lds_red[2][kWaves];
    __shared__ BatchCtl ctl;
    __shared__ ProbState st;
    const bool whole = ONE || stamp == 0;
    const double *__restrict__ X = A.X;
    double *out = P.out;
    if (whole) P.out = nullptr;   // stored at the end
    GridBarrier grid(A.sync);
    if (whole) {
        if (threadIdx.x < kWave) begin_problem(0, BEGIN_SOLVE, d, A.w0, A.C, &ctl, &st);
        if (blockIdx.x != 0) A.trace = nullptr;
    } else {
        copy_words(&ctl, A.ctl);
        copy_words(&st, A.st);
    }
    __syncthreads();
    using T = Tile<E, L, U, VEC>;
    constexpr bool kAhead = !ONE && svm && tiles_at_once(E, L, true) == 1;
    const TileWalk walk((n + T::RT - 1) / T::RT, kWaves, true);
    OneTile<E, L, U, VEC, LOSS> mine;
    if constexpr (ONE) mine.load(n, d, X, A.y);
    extern __shared__ __align__(16) double stream_lds[];
    TileStream<E, L, U, VEC> stream(STREAM ? stream_lds : nullptr, d);
    // the wavefront's first tile, asked for ahead
    auto first_tile = [&]() {
        if (!kAhead || walk.first >= walk.last) return;
        if (STREAM) stream.ask(X, n, d, walk.first, true);
        else T::load(X, n, d, walk.first * T::RT, threadIdx.x & (kWave - 1), mine.x);
    };
    if (whole) first_tile();
    bool done = false;
    for (int64_t round = 1;; ++round) {
        const int mode = __builtin_amdgcn_readfirstlane(ctl.mode[0]);
        if (mode == MODE_IDLE) {
            done = true;
            break;
        }
        void *D = __builtin_amdgcn_readfirstlane(ctl.dslot[0]) ? A.D[1] : A.D[0];
        const double *vec = ctl.vec[0];
        const int64_t at = (round & 1) * A.round_stride;
        double *partials = A.partials + at, *loss_partials = A.loss_partials + at;
        if constexpr (ONE) mine.pass(lds, lds_red, mode == MODE_FG, ctl.dslot[0], d, vec, D, partials, loss_partials);
        else if constexpr (kAhead) {
            uint64_t *words = static_cast<uint64_t *>(D);
            svm_solve_pass<E, L, U, VEC, STREAM>(lds, lds_red, mode == MODE_FG, n, d, X, A.y, vec, words, partials, loss_partials, mine.x, whole, stream);
        } else if (mode == MODE_FG) fun_grad_pass<E, L, U, VEC, LOSS, STREAM>(lds, lds_red, n, d, X, A.y, vec, D, partials, loss_partials, nullptr, stream_lds);
        else hv_pass<E, L, U, VEC, svm, false, svm, STREAM, true>(lds, n, d, X, D, vec, partials, stream_lds);
        if (whole) {
            grid.arrive();
            first_tile();
            if (!grid.wait()) break;
        } else if (!last_workgroup(A.ticket)) {
            return;
        }
        double col, loss, active;
        // (the rows with D != 0 are not counted here)
        if (dense_add_rows<kWaves>(lds, (int)gridDim.x, (int)d, partials, mode == MODE_FG ? loss_partials : nullptr, nullptr, col, loss, active))
            advance_problem(0, mode, d, col, loss, &ctl, &st, P, A.trace, whole ? nullptr : A.host, stamp);
        __syncthreads();
        if (!whole) {
            copy_words(A.ctl, &ctl);
            copy_words(A.st, &st);
            if (threadIdx.x == 0) *A.ticket = 0u;
            return;
        }
    }
    if (whole) {
        if (done && blockIdx.x == 0 && threadIdx.x < kWave) {
            // the host goes on when it sees this: everything that the call returns has arrived by then
            const int lane = threadIdx.x;
            if (lane < d) store_shared(out + lane, st.w[lane]);
            if (lane == 0) A.host->sc[0] = st.sc;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) __hip_atomic_store(&A.host->finished, (int64_t)1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        grid.leave();
    } else if (blockIdx.x == 0 && threadIdx.x < kWave)   // the solve ended in an earlier round
        advance_problem(0, MODE_IDLE, d, 0.0, 0.0, &ctl, &st, P, A.trace, A.host, stamp);
}

// ------------------------------------------------------------------ second stage of the wide matrices
// out[c] = add[c] + C * sum_b partials[b * d + c] and the scalars (see DenseFinish) for d > 32.  A workgroup takes 16
// columns; a wavefront reads four rows of partial sums (128 bytes each) per load, sixteen loads in flight, wavefront k the
// rows 4 k .. 4 k + 3 of every 64.  The scalars are sums over the columns, so the workgroup that finishes last adds up
// what the others left; it replaces a launch.  With one wavefront per column and its loads not batched this took 10 us for
// 2048 workgroups of 257 columns, and the scalars another 4 us.
__global__ __launch_bounds__(kColumnsBlock) void k_dense_columns(int d, int grid, const double *__restrict__ partials, double *__restrict__ col_partials,
                                                               const double *__restrict__ loss_partials, const double *__restrict__ active_partials,
                                                               DenseFinish fin)
{
    constexpr int kWaves = kColumnsBlock / kWave, kAtOnce = 16, kRows = kColumnsBlock / kColumnsPer;
    __shared__ double part[kWaves][kColumnsPer];
    __shared__ double red[4][kWaves];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int c = blockIdx.x * kColumnsPer + lane % kColumnsPer;
    double s = 0.0;
    for (int b0 = threadIdx.x / kColumnsPer; b0 < grid; b0 += kAtOnce * kRows) {
        double t[kAtOnce];
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k) {
            const int b = b0 + k * kRows;
            t[k] = (b < grid && c < d) ? partials[(int64_t)b * d + c] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k) s += t[k];
    }
    s = add_halves(add_row_pairs(s));   // the four rows of a load
    if (lane < kColumnsPer) part[wv][lane] = s;
    __syncthreads();
    if (wv == 0) {   // the outputs of the 16 columns, and what they add to the scalars
        double cp = 0.0, ww = 0.0;
        if (lane < kColumnsPer && c < d) {
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < kWaves; ++k) t += part[k][lane];
            const double add = fin.add ? fin.add[c] : 1.0;
            const double o = fma(fin.C, t, add);
            cp = o * (fin.dotw ? fin.dotw[c] : o);
            ww = add * add;
            if (fin.out) store_shared(fin.out + c, o);   // on its way before the ticket is drawn
        }
        cp = wave_sum(cp);
        ww = wave_sum(ww);
        if (fin.scal && lane == 0) {
            store_shared(col_partials + 2 * blockIdx.x, cp);
            store_shared(col_partials + 2 * blockIdx.x + 1, ww);
        }
    }
    if (!fin.scal || !last_workgroup(fin.ticket)) return;
    double v[4] = {0.0, 0.0, 0.0, 0.0};   // loss, w.w, sum of the column products, active rows
    if (fin.fun_grad)
        for (int b = threadIdx.x; b < grid; b += kColumnsBlock) {
            v[0] += loss_partials[b];
            v[3] += active_partials[b];
        }
    if (threadIdx.x < gridDim.x) {
        v[2] = load_shared(col_partials + 2 * threadIdx.x);
        v[1] = load_shared(col_partials + 2 * threadIdx.x + 1);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = wave_sum(v[k]);
        if (lane == 0) red[k][wv] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t[4] = {0.0, 0.0, 0.0, 0.0};
        for (int k = 0; k < 4; ++k)
            for (int m = 0; m < kWaves; ++m) t[k] += red[k][m];
        store_dense_scalars(fin, t[0], t[1], t[2], t[3]);
        *fin.ticket = 0u;
    }
    if (threadIdx.x < kWave) post_flag(fin.flag);
}

// ------------------------------------------------------------------ dispatch
constexpr double kSkipBelow = 0.95;   // active fraction under which the Hessian-vector pass skips the inactive rows

// A row that is left out saves bytes only if nothing else of its 128-byte lines is read.  For rows shorter than a line the pass
// skips where at least a tenth of the lines is free of active rows, (1 - active)^(rows per line) >= 0.1.  L2-SVM calls, every
// row read by 256 workgroups / the better of skipping with 256 and 512: 20M x 1, 0.2 of the rows active 40 / 43 us, 0.05
// 40 / 38; 20M x 3, 0.5 91 / 91 (256: 125), 0.2 91 / 84; 16M x 5, 0.5 116 / 118 (256: 173), 0.2 116 / 108; 10M x 8, 0.85
// 120 / 118 (256: 133), 0.5 115 / 95; 8M x 12, 0.94 141 / 142, 0.7 139 / 128; 6M x 16, 0.85 143 / 129.
constexpr int kLineDoubles = 16;
constexpr double kFreeLines = 0.1;

// Where about half of the rows or fewer are read, the loads that are left out no longer fill the queue to HBM with eight
// wavefronts per CU: d <= 32 then runs two workgroups per CU.  20M x 24, 256 / 512 workgroups: 0.72 of the rows active 490 / 503
// us, 0.47 364 / 358, 0.38 335 / 294, 0.36 330 / 281.  Rows of a line or less gain at any fraction that is skipped once the
// pass is long: 10M x 8, 0.7 active 127 / 112, 6M x 16, 0.85 133 / 129, 0.5 97 / 82; but 3M x 12, 0.5 48 / 49.  Below 2M rows the
// additional tickets cost more: 1M x 24, 0.35 31 / 34, 1M x 8, 0.2 25 / 27, 200,000 x 4, 0.2 20 / 22 (2M x 24, 0.2 40 / 37).
constexpr double kFewBelow = 0.5;
constexpr int64_t kFewRows = 2'000'000, kFewShortRows = 6'000'000;

bool skip_pays(int64_t d, double active)
{
    if (d >= kLineDoubles) return active < kSkipBelow;
    return std::pow(std::max(0.0, 1.0 - active), (double)kLineDoubles / (double)d) >= kFreeLines;
}

bool few_active(int64_t n, int64_t d, double active)
{
    return d <= kFinishMaxD && n >= kFewRows && (active < kFewBelow || (d <= kLineDoubles && n >= kFewShortRows));
}

// What a Hessian-vector pass runs over: the matrix itself with D of one buffer, or the compacted copy of its active rows
// (then every row is active: the bit words are all ones).
struct HvInput {
    const double *X;
    int64_t n;
    const void *D;
    bool mask, skip;
    int grid;
};

HvInput hv_input(const tron_dataset *ds, int Dslot)
{
    if (ds->hat_slot == Dslot && ds->Xhat)
        return HvInput{ds->Xhat, ds->hat_rows, ds->hat_bits, true, false, dense_grid_for(ds->hat_rows, ds->d)};
    const double active = ds->active_frac[Dslot];
    const bool mask = ds->D_is_mask[Dslot], skip = mask && skip_pays(ds->d, active);
    const bool few = skip && few_active(ds->n, ds->d, active);
    return HvInput{ds->X, ds->n, ds->Dbuf[Dslot], mask, skip, few ? dense_grid_few(ds->n, ds->d) : ds->dense_grid};
}

// Workgroups that read X through LDS want more of it than the 64 KB that a launch has without asking
template <auto Kernel>
int allow_lds(int bytes)
{
    static std::atomic<uint64_t> asked{0};   // a bit per device
    int dev = 0;
    if (bytes <= 64 << 10) return TRON_OK;
    TRON_HIP(hipGetDevice(&dev));
    const uint64_t bit = 1ull << (dev & 63);
    if (asked.load(std::memory_order_relaxed) & bit) return TRON_OK;
    TRON_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)TileStream<8, 4, 4, true>::bytes(kFinishMaxD, dense_block(4) / kWave)));
    asked.fetch_or(bit, std::memory_order_relaxed);
    return TRON_OK;
}

// bytes of LDS through which a pass reads X
template <int L>
int stream_bytes(int64_t n, int64_t d) { return tiles_stream(L) && read_once(n, d) ? (int)(512 * d * (dense_block(L) / kWave)) : 0; }

template <int E, int L>
int launch_hv(tron_dataset *ds, const HvInput &in, const double *v, double *partials, const DenseFinish &fin)
{
    constexpr int U = pick_U(E, L);
    const bool vec = (E % 2 == 0) && (ds->d % 2 == 0);
    const int grid = in.grid;
    const void *D = in.D;
    const bool mask = in.mask, skip = in.skip;
    const int through = skip && mask ? 0 : stream_bytes<L>(in.n, ds->d);
#define TRON_HV_T(V, M, G, S, T) do { \
        TRON_TRY((allow_lds<k_dense_hv<E, L, U, V, M, G, S, T>>(through))); \
        hipLaunchKernelGGL((k_dense_hv<E, L, U, V, M, G, S, T>), dim3(grid), dim3(dense_block(L)), through, ds->stream, in.n, ds->d, in.X, D, v, partials, fin); \
    } while (0)
#define TRON_HV(V, M, G, S) do { if (through) TRON_HV_T(V, M, G, S, (tiles_stream(L) && !S)); else TRON_HV_T(V, M, G, S, false); } while (0)
#define TRON_HV_V(M, G, S) do { if (vec) TRON_HV((E % 2 == 0), M, G, S); else TRON_HV(false, M, G, S); } while (0)
    if (v) {
        if (!mask) TRON_HV_V(false, false, false);
        else if (skip) TRON_HV_V(true, false, true);
        else TRON_HV_V(true, false, false);
    } else {   // no vector: the diagonal sums
        if (!mask) TRON_HV_V(false, true, false);
        else if (skip) TRON_HV_V(true, true, true);
        else TRON_HV_V(true, true, false);
    }
#undef TRON_HV_V
#undef TRON_HV
#undef TRON_HV_T
    return TRON_OK;
}

template <int E, int L>
int launch_fg(tron_dataset *ds, int loss, const double *w, void *Dout, double *loss_partials, double *active_partials, const DenseFinish &fin)
{
    constexpr int U = pick_U(E, L);
    const bool vec = (E % 2 == 0) && (ds->d % 2 == 0);
    const int grid = dense_fun_grad_grid(ds->n, ds->d);
    const int through = stream_bytes<L>(ds->n, ds->d);
#define TRON_FG_T(V, LS, T) do { \
        TRON_TRY((allow_lds<k_dense_fun_grad<E, L, U, V, LS, T>>(through))); \
        hipLaunchKernelGGL((k_dense_fun_grad<E, L, U, V, LS, T>), dim3(grid), dim3(dense_block(L)), through, ds->stream, ds->n, ds->d, ds->X, ds->y8, w, Dout, ds->partials, loss_partials, active_partials, fin); \
    } while (0)
#define TRON_FG(V, LS) do { if (through) TRON_FG_T(V, LS, tiles_stream(L)); else TRON_FG_T(V, LS, false); } while (0)
    if (loss == TRON_LOSS_LR) {
        if (vec) TRON_FG((E % 2 == 0), TRON_LOSS_LR); else TRON_FG(false, TRON_LOSS_LR);
    } else {
        if (vec) TRON_FG((E % 2 == 0), TRON_LOSS_L2SVM); else TRON_FG(false, TRON_LOSS_L2SVM);
    }
#undef TRON_FG
#undef TRON_FG_T
    return TRON_OK;
}

template <int E, int L>
int launch_solve(tron_dataset *ds, const SolveParams &P, const SolveArgs &A, int64_t stamp)
{
    if constexpr (dense_finishes(L)) {
        constexpr int U = pick_U(E, L);
        const bool vec = (E % 2 == 0) && (ds->d % 2 == 0);
        const int grid = dense_round_grid(ds->n, ds->d, P.loss);
        const bool one = stamp == 0 && (ds->n + kWave - 1) / kWave <= (int64_t)grid * (dense_block(L) / kWave);
        const int through = stream_bytes<L>(ds->n, ds->d);
#define TRON_SOLVE_T(V, LS, R) do { \
        TRON_TRY((allow_lds<k_dense_solve<E, L, U, V, LS, R>>(through))); \
        hipLaunchKernelGGL((k_dense_solve<E, L, U, V, LS, R>), dim3(grid), dim3(dense_block(L)), through, ds->stream, ds->n, ds->d, A, P, stamp); \
    } while (0)
#define TRON_SOLVE(V, LS) do { \
        if (one) TRON_SOLVE_T(V, LS, ROWS_KEPT); \
        else if (through) TRON_SOLVE_T(V, LS, (tiles_stream(L) ? ROWS_STREAMED : ROWS_LOADED)); \
        else TRON_SOLVE_T(V, LS, ROWS_LOADED); \
    } while (0)
        if (P.loss == TRON_LOSS_LR) {
            if (vec) TRON_SOLVE((E % 2 == 0), TRON_LOSS_LR); else TRON_SOLVE(false, TRON_LOSS_LR);
        } else {
            if (vec) TRON_SOLVE((E % 2 == 0), TRON_LOSS_L2SVM); else TRON_SOLVE(false, TRON_LOSS_L2SVM);
        }
#undef TRON_SOLVE
#undef TRON_SOLVE_T
        TRON_HIP(hipGetLastError());
        return TRON_OK;
    } else {
        set_error("internal: a solve driven from the device needs d <= %d", kFinishMaxD);
        return TRON_EINVAL;
    }
}

// E in 1..8 for L = 1, E in 5..8 for L >= 2 (smaller d picks a smaller L)
#define TRON_DISPATCH_E(L_, FN, ...)                         \
    switch (s.E) {                                           \
    case 5: return FN<5, L_>(__VA_ARGS__);                   \
    case 6: return FN<6, L_>(__VA_ARGS__);                   \
    case 7: return FN<7, L_>(__VA_ARGS__);                   \
    case 8: return FN<8, L_>(__VA_ARGS__);                   \
    default: break;                                          \
    }

#define TRON_DISPATCH(FN, ...)                                                   \
    Shape s;                                                                     \
    if (!pick_shape(ds->d, s)) { set_error("dense d = %lld not supported (max 512)", (long long)ds->d); return TRON_EINVAL; } \
    switch (s.L) {                                                               \
    case 1:                                                                      \
        switch (s.E) {                                                           \
        case 1: return FN<1, 1>(__VA_ARGS__);                                    \
        case 2: return FN<2, 1>(__VA_ARGS__);                                    \
        case 3: return FN<3, 1>(__VA_ARGS__);                                    \
        case 4: return FN<4, 1>(__VA_ARGS__);                                    \
        default: break;                                                          \
        }                                                                        \
        TRON_DISPATCH_E(1, FN, __VA_ARGS__) break;                               \
    case 2: TRON_DISPATCH_E(2, FN, __VA_ARGS__) break;                           \
    case 4: TRON_DISPATCH_E(4, FN, __VA_ARGS__) break;                           \
    case 8: TRON_DISPATCH_E(8, FN, __VA_ARGS__) break;                           \
    case 16: TRON_DISPATCH_E(16, FN, __VA_ARGS__) break;                         \
    case 32: TRON_DISPATCH_E(32, FN, __VA_ARGS__) break;                         \
    case 64: TRON_DISPATCH_E(64, FN, __VA_ARGS__) break;                         \
    default: break;                                                              \
    }                                                                            \
    set_error("internal: no dense kernel for E=%d L=%d", s.E, s.L);              \
    return TRON_EINVAL;

int dispatch_hv(tron_dataset *ds, const HvInput &in, const double *v, double *partials, const DenseFinish &fin) { TRON_DISPATCH(launch_hv, ds, in, v, partials, fin) }
int dispatch_fg(tron_dataset *ds, int loss, const double *w, void *Dout, double *lp, double *ap, const DenseFinish &fin) { TRON_DISPATCH(launch_fg, ds, loss, w, Dout, lp, ap, fin) }
int dispatch_solve(tron_dataset *ds, const SolveParams &P, const SolveArgs &A, int64_t stamp) { TRON_DISPATCH(launch_solve, ds, P, A, stamp) }

// the second stage of a wide matrix; the others have completed it in the pass
int launch_columns(tron_dataset *ds, int grid, const double *partials, double *col_partials, const double *loss_partials, const double *active_partials,
                   const DenseFinish &fin)
{
    if (ds->d <= kFinishMaxD) return TRON_OK;
    ProfScope ps(ds, SLOT_DENSE_FINALIZE);
    hipLaunchKernelGGL(k_dense_columns, dim3((unsigned)((ds->d + kColumnsPer - 1) / kColumnsPer)), dim3(kColumnsBlock), 0, ds->stream, (int)ds->d, grid,
                       partials, col_partials, loss_partials, active_partials, fin);
    TRON_HIP(hipGetLastError());
    return TRON_OK;
}

}  // namespace

__global__ __launch_bounds__(kBlock) void k_labels_to_int8(int64_t m, const double *__restrict__ y, int8_t *__restrict__ y8)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m; i += (int64_t)gridDim.x * kBlock)
        y8[i] = (y[i] > 0.0) ? 1 : -1;
}

// Input check for rows handed over in device memory: flag[0] = 1 when a label is not exactly +1 or -1, flag[1] = 1 when
// an entry of X is not finite (every offending thread stores the same value).
__global__ __launch_bounds__(kBlock) void k_dense_validate(int64_t m, int64_t count, const double *__restrict__ X,
                                                           const double *__restrict__ y, double *__restrict__ flag)
{
    const int64_t t0 = (int64_t)blockIdx.x * kBlock + threadIdx.x, stride = (int64_t)gridDim.x * kBlock;
    bool bad_y = false, bad_x = false;
    for (int64_t i = t0; i < m; i += stride) bad_y |= !(y[i] == 1.0 || y[i] == -1.0);
    for (int64_t k = t0; k < count; k += stride) bad_x |= !isfinite(X[k]);
    if (bad_y) flag[0] = 1.0;
    if (bad_x) flag[1] = 1.0;
}

// what: 0 = fine, 1 = a label is not +1 / -1, 2 = a matrix entry is not finite.  Synchronises the stream.
int dense_validate_device(tron_dataset *ds, int64_t m, const double *X_dev, const double *y_dev, int *what)
{
    double *flag_host = ds->scal_host + kScalars - 2;   // the last two scalar slots: written by no other kernel
    flag_host[0] = 0.0;
    flag_host[1] = 0.0;
    int64_t g = (m * ds->d + kBlock * 8 - 1) / (kBlock * 8);
    if (g < 1) g = 1;
    if (g > kMaxGrid) g = kMaxGrid;
    hipLaunchKernelGGL(k_dense_validate, dim3((int)g), dim3(kBlock), 0, ds->stream, m, m * ds->d, X_dev, y_dev, ds->scal_dev + kScalars - 2);
    TRON_HIP(hipGetLastError());
    TRON_HIP(hipStreamSynchronize(ds->stream));
    *what = flag_host[0] != 0.0 ? 1 : (flag_host[1] != 0.0 ? 2 : 0);
    return TRON_OK;
}

int dense_labels_from_device(tron_dataset *ds, int64_t row0, int64_t m, const double *y_dev)
{
    int64_t g = (m + kBlock - 1) / kBlock;
    if (g > kMaxGrid) g = kMaxGrid;
    hipLaunchKernelGGL(k_labels_to_int8, dim3((int)g), dim3(kBlock), 0, ds->stream, m, y_dev, ds->y8 + row0);
    TRON_HIP(hipGetLastError());
    return TRON_OK;
}

// ------------------------------------------------------------------ compacted copy of the active rows
// Section 5 of the paper keeps X_hat = X_{I,:} in device memory so that its matrix-vector products touch active rows
// only.  Here the copy is optional (the Hessian-vector pass over X skips inactive rows by itself): it pays when many
// products follow at one iterate with a small active set, because a pass over contiguous rows streams faster than one
// that picks 192-byte rows out of X.  Built on the device from the bit words the function/gradient pass left:
//   1. active rows before every 64-row tile: popcounts, scanned in three steps (per workgroup, over the workgroups, back);
//   2. every wavefront copies the active rows of its tiles to their places in X_hat (reads of inactive rows are not issued);
//   3. the active set of the copy is all ones.
constexpr int kScanPer = 4;                                   // tiles per thread in the scan
constexpr int kScanTile = kBlock * kScanPer;                  // tiles per workgroup

__global__ __launch_bounds__(kBlock) void k_active_block_sums(int64_t ntiles, const uint64_t *__restrict__ bits, int64_t *__restrict__ block_sums)
{
    __shared__ double lds[kWavesPerBlock];
    const int64_t t0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanPer;
    int c = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k)
        if (t0 + k < ntiles) c += __popcll(bits[t0 + k]);
    const double s = block_sum((double)c, lds);   // exact: at most 2^18 per workgroup
    if (threadIdx.x == 0) block_sums[blockIdx.x] = (int64_t)s;
}

// exclusive scan of the workgroup sums, in place, by one workgroup (thread t owns a contiguous run of them)
__global__ __launch_bounds__(kBlock) void k_active_scan_blocks(int nblocks, int64_t *__restrict__ block_sums)
{
    __shared__ int64_t run[kBlock];
    const int per = (nblocks + kBlock - 1) / kBlock;
    const int b0 = threadIdx.x * per, b1 = (b0 + per < nblocks) ? b0 + per : nblocks;
    int64_t s = 0;
    for (int b = b0; b < b1; ++b) s += block_sums[b];
    run[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t acc = 0;
        for (int t = 0; t < kBlock; ++t) { const int64_t v = run[t]; run[t] = acc; acc += v; }
    }
    __syncthreads();
    int64_t acc = run[threadIdx.x];
    for (int b = b0; b < b1; ++b) { const int64_t v = block_sums[b]; block_sums[b] = acc; acc += v; }
}

__global__ __launch_bounds__(kBlock) void k_active_tile_offsets(int64_t ntiles, const uint64_t *__restrict__ bits,
                                                                const int64_t *__restrict__ block_sums, int64_t *__restrict__ tile_off)
{
    __shared__ int wave_tot[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int64_t t0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanPer;
    int c[kScanPer], mine = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        c[k] = (t0 + k < ntiles) ? __popcll(bits[t0 + k]) : 0;
        mine += c[k];
    }
    const int incl = wave_scan_add(mine);
    if (lane == kWave - 1) wave_tot[wv] = incl;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wv; ++w) before += wave_tot[w];
    int64_t off = block_sums[blockIdx.x] + before + incl - mine;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        if (t0 + k < ntiles) tile_off[t0 + k] = off;
        off += c[k];
    }
}

// VEC: d is even, rows are moved in 16-byte pieces
template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_compact_rows(int64_t n, int d, uint64_t inv_d, const double *__restrict__ X,
                                                         const uint64_t *__restrict__ bits, const int64_t *__restrict__ tile_off,
                                                         double *__restrict__ Xhat)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t ntiles = (n + kWave - 1) / kWave;
    const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
    constexpr int W = VEC ? 2 : 1;
    for (int64_t tile = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave; tile < ntiles; tile += nwaves) {
        const uint64_t b = bits[tile];   // rows past n are never set
        if (b == 0) continue;
        const double *src = X + tile * kWave * d;
        double *dst = Xhat + tile_off[tile] * d;
        const int total = kWave * d;
        for (int e = lane * W; e < total; e += kWave * W) {
            const int row = (int)(((uint64_t)e * inv_d) >> 32);   // e / d, exact for e < 64 * 32 (inv_d = ceil(2^32 / d))
            if ((b >> row) & 1u) {
                const int rank = __popcll(b & ((1ull << row) - 1ull));
                const int col = e - row * d;
                if (VEC) *reinterpret_cast<double2 *>(dst + rank * d + col) = *reinterpret_cast<const double2 *>(src + e);
                else dst[rank * d + col] = src[e];
            }
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_all_active_bits(int64_t rows, uint64_t *__restrict__ bits)
{
    const int64_t words = (rows + kWave - 1) / kWave;
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < words; t += (int64_t)gridDim.x * kBlock) {
        const int64_t left = rows - t * kWave;
        bits[t] = (left >= kWave) ? ~0ull : ((1ull << left) - 1ull);
    }
}

bool dense_compact_wanted(const tron_dataset *ds, int Dslot, int recent_cg_iters)
{
    if (!ds->dense || ds->d > 32 || !ds->D_is_mask[Dslot] || g_tuning.dense_compact == 0) return false;
    if (ds->active_count[Dslot] <= 0 || ds->active_frac[Dslot] >= kSkipBelow) return false;
    if (g_tuning.dense_compact > 0) return true;
    // Building the copy costs as much as 2.8 products over it, and a product over it saves about a fifth of the row-skipping
    // one: paid for after 11 to 13 products per iterate at 0.36 to 0.47 of the rows active, 26 at 0.72 (20M x 24).  The
    // inner solve before had ten or more: the next one, nearer the solution, tends to be longer.
    return ds->active_frac[Dslot] <= 0.6 && recent_cg_iters >= 10;
}

int dense_compact_build(tron_dataset *ds, int Dslot)
{
    if (!ds->dense || ds->d > 32 || !ds->D_is_mask[Dslot]) { set_error("internal: no bit-word active set to compact"); return TRON_EINVAL; }
    const int64_t rows = ds->active_count[Dslot];
    const int64_t ntiles = (ds->n + kWave - 1) / kWave;
    const int nblocks = (int)((ntiles + kScanTile - 1) / kScanTile);
    ds->hat_slot = -1;
    if (!ds->tile_off) {
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->tile_off), sizeof(int64_t) * (size_t)(ntiles + 1)));
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->scan_blocks), sizeof(int64_t) * (size_t)(nblocks + 1)));
    }
    if (rows > ds->hat_cap) {
        // grow with some room, so that a slowly growing active set does not reallocate at every iterate
        TRON_HIP(hipStreamSynchronize(ds->stream));
        hipFree(ds->Xhat); hipFree(ds->hat_bits);
        ds->Xhat = nullptr; ds->hat_bits = nullptr; ds->hat_cap = 0;
        int64_t cap = rows + rows / 8 + 1024;
        if (cap > ds->n) cap = ds->n;
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->Xhat), sizeof(double) * (size_t)cap * (size_t)ds->d));
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ds->hat_bits), sizeof(uint64_t) * (size_t)(cap / kWave + 1)));
        ds->hat_cap = cap;
    }
    ProfScope ps(ds, SLOT_DENSE_COMPACT);
    const uint64_t *bits = static_cast<const uint64_t *>(static_cast<const void *>(ds->Dbuf[Dslot]));
    hipLaunchKernelGGL(k_active_block_sums, dim3(nblocks), dim3(kBlock), 0, ds->stream, ntiles, bits, ds->scan_blocks);
    hipLaunchKernelGGL(k_active_scan_blocks, dim3(1), dim3(kBlock), 0, ds->stream, nblocks, ds->scan_blocks);
    hipLaunchKernelGGL(k_active_tile_offsets, dim3(nblocks), dim3(kBlock), 0, ds->stream, ntiles, bits, ds->scan_blocks, ds->tile_off);
    int64_t g = (ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
    if (g > kMaxGrid) g = kMaxGrid;
    const uint64_t inv_d = ((1ull << 32) + (uint64_t)ds->d - 1) / (uint64_t)ds->d;
    if (ds->d % 2 == 0)
        hipLaunchKernelGGL(k_compact_rows<true>, dim3((int)g), dim3(kBlock), 0, ds->stream, ds->n, ds->d, inv_d, ds->X, bits, ds->tile_off, ds->Xhat);
    else
        hipLaunchKernelGGL(k_compact_rows<false>, dim3((int)g), dim3(kBlock), 0, ds->stream, ds->n, ds->d, inv_d, ds->X, bits, ds->tile_off, ds->Xhat);
    const int64_t words = (rows + kWave - 1) / kWave;
    int64_t gb = (words + kBlock - 1) / kBlock;
    if (gb < 1) gb = 1;
    if (gb > kMaxGrid) gb = kMaxGrid;
    hipLaunchKernelGGL(k_all_active_bits, dim3((int)gb), dim3(kBlock), 0, ds->stream, rows, ds->hat_bits);
    TRON_HIP(hipGetLastError());
    ds->hat_rows = rows;
    ds->hat_slot = Dslot;
    return TRON_OK;
}

void dense_compact_release(tron_dataset *ds)
{
    hipFree(ds->Xhat); hipFree(ds->hat_bits); hipFree(ds->tile_off); hipFree(ds->scan_blocks);
    ds->Xhat = nullptr; ds->hat_bits = nullptr; ds->tile_off = nullptr; ds->scan_blocks = nullptr;
    ds->hat_cap = ds->hat_rows = 0;
    ds->hat_slot = -1;
}

bool dense_supported(int64_t d)
{
    Shape s;
    return d >= 1 && pick_shape(d, s);
}

static int grid_up_to(int64_t n, int64_t d, int64_t most)
{
    Shape s;
    if (!pick_shape(d, s)) return 1;
    const int64_t rows = (int64_t)pick_U(s.E, s.L) * (kWave / s.L) * (dense_block(s.L) / kWave);
    const int64_t g = (n + rows - 1) / rows;
    return (int)(g < most ? g : most);
}

int dense_grid_for(int64_t n, int64_t d) { return grid_up_to(n, d, d <= kFinishMaxD ? kFinishGrid : kWideGrid); }
int dense_grid_few(int64_t n, int64_t d) { return grid_up_to(n, d, kFewGrid); }

// A function/gradient pass over narrow rows is bound by the chain of operations of a tile, not by its bytes, so what helps is
// more wavefronts; their tickets (10 ns each) pay from some millions of rows on, in the rounds of a solve, where the Hessian-vector
// passes pay them too, later than in calls.  Calls with 256 / 512 workgroups: 20M rows, d = 1 L2-SVM 88 / 58 us, logistic
// 169 / 121; d = 4 155 / 133 and 192 / 174; d = 5 L2-SVM 187 / 161, logistic 214 / 212, 6M rows 74 / 64 (the logistic rounds
// lose by it: 20M x 5 1007 / 1032 us a solve); 4M x 3 37 / 36 and 45 / 41, 4M x 4 38 / 40 and 45 / 42; 2M x 2 25 / 26 and
// 32 / 31.  512 / 1024, 20M rows, L2-SVM: d = 1 58 / 52, d = 2 86 / 77, d = 3 105 / 114; a solve's rounds, 40M x 2: 450 / 472.
// The Hessian-vector rounds of the L2-SVM leave out inactive rows whatever their number, whose loads want 512 workgroups up to
// d = 8: solves with 256 / 512, (nearly) all rows active and few, 20M x 6 1020 / 872 and 1804 / 1450 us, 6M x 6 320 / 302
// and 543 / 493, 16M x 7 953 / 922 and 1655 / 1600, 15M x 8 932 / 929 and 1597 / 1495; 6M x 9 466 / 478 and 763 / 757, 8M x 13
// 827 / 1007 and 1335 / 1550.
constexpr int64_t kNarrowRows = 6'000'000, kNarrowCallRows = 3'000'000, kNarrowestRows = 16'000'000;
constexpr int kNarrowGrid = 512, kNarrowestGrid = 1024;

int dense_round_grid(int64_t n, int64_t d, int loss)
{
    const bool narrow = d <= 4 || (d <= 8 && loss == TRON_LOSS_L2SVM);
    return narrow && n >= kNarrowRows ? grid_up_to(n, d, kNarrowGrid) : dense_grid_for(n, d);
}

int dense_fun_grad_grid(int64_t n, int64_t d)
{
    if (d <= 2 && n >= kNarrowestRows) return grid_up_to(n, d, kNarrowestGrid);
    if ((d <= 3 && n >= kNarrowCallRows) || (d <= 5 && n >= kNarrowRows)) return grid_up_to(n, d, kNarrowGrid);
    return dense_grid_for(n, d);
}

int dense_work_units(int64_t n, int64_t d)
{
    Shape s;
    if (!pick_shape(d, s)) return 1;
    const int64_t rows = (int64_t)pick_U(s.E, s.L) * (kWave / s.L) * kWavesPerBlock;
    const int64_t g = (n + rows - 1) / rows;
    return (int)(g > kMaxGrid ? kMaxGrid : g);
}

// column sums (grid * d) followed by loss partials (grid), the column workgroups' sums (d) and active-row counts (grid); a solve
// driven from the device has two sets of sums
int64_t dense_partials_needed(int64_t n, int64_t d)
{
    int64_t g = d <= kFinishMaxD ? dense_grid_few(n, d) : dense_grid_for(n, d);   // the largest grid of a pass
    g = std::max<int64_t>(g, dense_fun_grad_grid(n, d));
    for (int loss : {TRON_LOSS_LR, TRON_LOSS_L2SVM}) g = std::max<int64_t>(g, dense_round_grid(n, d, loss));
    return (d <= kFinishMaxD ? 2 : 1) * (d * g + g + d + g);
}

// D of n rows as a pass keeps it: fp64, or the active set as one bit (d <= 32) or one byte a row
static int64_t d_bytes(int64_t n, int64_t d, bool mask) { return !mask ? 8 * n : (d <= kFinishMaxD ? n / 8 : n); }

int64_t dense_hv_bytes(const tron_dataset *ds)
{
    if (!ds->have_D) return 8 * ds->n * ds->d + d_bytes(ds->n, ds->d, false) + 8 * ds->d * ds->dense_grid;
    const HvInput in = hv_input(ds, ds->Dcur);
    const double frac = (in.skip && ds->d <= kFinishMaxD) ? ds->active_frac[ds->Dcur] : 1.0;   // the bytes of wider rows are all read
    return (int64_t)(8.0 * frac * (double)in.n * (double)ds->d) + d_bytes(in.n, ds->d, in.mask) + 8 * ds->d * in.grid;
}

int64_t dense_fun_grad_bytes(const tron_dataset *ds)
{
    const bool mask = ds->have_D && ds->D_is_mask[ds->Dcur];
    const int grid = dense_fun_grad_grid(ds->n, ds->d);
    return 8 * ds->n * ds->d + ds->n + d_bytes(ds->n, ds->d, mask) + 8 * ds->d * grid;
}

int dense_hv(tron_dataset *ds, double C, int Dslot, const double *v, double *Hv)
{
    const HvInput in = hv_input(ds, Dslot);
    const DenseFinish fin{ds->ticket, v, C, Hv, v, ds->scal_dev, ds->scal_copy, false, next_flag(ds)};
    {
        ProfScope ps(ds, SLOT_DENSE_HV);
        TRON_TRY(dispatch_hv(ds, in, v, ds->partials, fin));
        TRON_HIP(hipGetLastError());
    }
    return launch_columns(ds, in.grid, ds->partials, ds->partials + (ds->d + 1) * ds->dense_grid, nullptr, nullptr, fin);
}

// out = 1 + C diag(X^T D X): the same pass as dense_hv with squared entries
int dense_hess_diag(tron_dataset *ds, double C, int Dslot, double *out)
{
    const HvInput in = hv_input(ds, Dslot);
    const DenseFinish fin{ds->ticket, nullptr, C, out, nullptr, nullptr, nullptr, false, HostFlag{nullptr, 0}};
    {
        ProfScope ps(ds, SLOT_DENSE_HV);
        TRON_TRY(dispatch_hv(ds, in, nullptr, ds->partials, fin));
        TRON_HIP(hipGetLastError());
    }
    return launch_columns(ds, in.grid, ds->partials, ds->partials + (ds->d + 1) * ds->dense_grid, nullptr, nullptr, fin);
}

int dense_solve_launch(tron_dataset *ds, const SolveParams &P, DriverState &drv, int64_t stamp, const double *w0, double C)
{
    const int grid = dense_round_grid(ds->n, ds->d, P.loss);
    double *loss_partials = ds->partials + ds->d * grid;
    const SolveArgs A{ds->X, ds->y8, {ds->Dbuf[0], ds->Dbuf[1]}, ds->partials, loss_partials, (ds->d + 1) * grid,
                      ds->ticket, grid_sync(ds), drv.ctl, drv.st, w0, C, P.trace_cap > 0 ? drv.trace_dev : nullptr, drv.host_dev};
    ProfScope ps(ds, SLOT_BATCH_PASS);
    return dispatch_solve(ds, P, A, stamp);
}

int dense_fun_grad(tron_dataset *ds, int loss, double C, const double *w, int Dslot, double *g)
{
    void *Dout = ds->Dbuf[Dslot];
    if (ds->hat_slot == Dslot) ds->hat_slot = -1;   // the compacted copy belonged to the D that is overwritten now
    ds->D_is_mask[Dslot] = (loss == TRON_LOSS_L2SVM);
    const int grid = dense_fun_grad_grid(ds->n, ds->d);
    double *loss_partials = ds->partials + ds->d * grid;
    double *col_partials = loss_partials + grid;
    double *active_partials = col_partials + ds->d;
    const DenseFinish fin{ds->ticket, w, C, g, nullptr, ds->scal_dev, ds->scal_copy, true, next_flag(ds)};
    {
        ProfScope ps(ds, SLOT_DENSE_FUN_GRAD);
        TRON_TRY(dispatch_fg(ds, loss, w, Dout, loss_partials, active_partials, fin));
        TRON_HIP(hipGetLastError());
    }
    return launch_columns(ds, grid, ds->partials, col_partials, loss_partials, active_partials, fin);
}

}  // namespace tron

// ------------------------------------------------------------------ Hessian-vector product without any allocation
// The work space of the dense Hessian-vector product -- per-workgroup column sums (d * grid), the column workgroups' sums (d),
// the curvature scalar and the counter of finished workgroups -- in a file-scope device object instead of the handle's
// allocation: a product enqueued here shares nothing that is written with the handle's own calls, so a captured one may be
// replayed beside them.  Every GPU the library runs on holds its own copy of the object, at its own address, until the
// process ends.
namespace {
constexpr int64_t kStaticScratchDoubles = TRON_HV_STATIC_MAX_DOUBLES;
struct StaticWork {
    double sums[kStaticScratchDoubles];
    unsigned ticket;
};
__device__ __align__(256) StaticWork static_work;
constexpr int kStaticMaxDevices = 64;
StaticWork *g_static_work[kStaticMaxDevices] = {nullptr};   // device address of `static_work` on each GPU, looked up once
}  // namespace

extern "C" int tron_hv_static(tron_dataset *ds, double C, const double *v_dev, double *Hv_dev, double *vHv_dev)
{
    using namespace tron;
    if (!ds || !v_dev || !Hv_dev || v_dev == Hv_dev || !(C > 0.0) || !std::isfinite(C)) {
        set_error("tron_hv_static: bad argument (null handle/v/Hv, v aliases Hv, or C <= 0)");
        return TRON_EINVAL;
    }
    if (!ds->dense) { set_error("tron_hv_static: dense handles only"); return TRON_EINVAL; }
    if (!ds->have_D) { set_error("tron_hv_static: no cached D; call tron_fun_grad first"); return TRON_ESTATE; }
    const int Dslot = ds->Dcur;
    const HvInput in = hv_input(ds, Dslot);
    const int grid = in.grid;
    // The limit is stated in groups of four wave tiles (dense_work_units); the sums of the workgroups that are launched, at most
    // 512 and never more than those groups, fit wherever it holds.
    const int units = dense_work_units(in.n, ds->d);
    const int64_t need = ds->d * units + ds->d + 1;
    if (need > kStaticScratchDoubles) {
        set_error("tron_hv_static: n = %lld, d = %lld needs %lld doubles of work space (d * %d groups of four wave tiles + d + 1); the static "
                  "work space holds %lld: use tron_hv", (long long)ds->n, (long long)ds->d, (long long)need, units,
                  (long long)kStaticScratchDoubles);
        return TRON_EINVAL;
    }
    int dev = -1;
    TRON_HIP(hipGetDevice(&dev));
    if (dev != ds->device || dev < 0 || dev >= kStaticMaxDevices) {
        set_error("tron_hv_static: current device %d is not the handle's device %d (or beyond %d devices)", dev, ds->device,
                  kStaticMaxDevices);
        return TRON_EINVAL;
    }
    if (!g_static_work[dev]) {
        // in host code the object's name is only a stand-in: its address on this GPU comes from the runtime
        StaticWork *p = nullptr;
        TRON_HIP(hipGetSymbolAddress(reinterpret_cast<void **>(&p), HIP_SYMBOL(static_work)));
        if (!p) { set_error("tron_hv_static: the static work space has no device address"); return TRON_EDEVICE; }
        g_static_work[dev] = p;
    }
    double *partials = g_static_work[dev]->sums;
    double *colprod = partials + ds->d * grid;
    double *scalar = colprod + ds->d;
    // Nothing has to start at zero: every workgroup of the pass writes all d of its column sums, the second stage the rest.  Calls
    // that overlapped (they race for the sums) spoil their own results and no later ones: for d <= 32 the sums are added by a
    // launch of its own, without a counter, for wider rows the pass clears the counter of k_dense_columns first.  (A counter in
    // the pass needs a launch that clears it: 20,003 x 8 then takes 21.1 us a call, this way 19.1.)
    const bool narrow = ds->d <= kFinishMaxD;
    const DenseFinish fin{narrow ? nullptr : &g_static_work[dev]->ticket, v_dev, C, Hv_dev, v_dev, vHv_dev ? vHv_dev : scalar, scalar, false, HostFlag{nullptr, 0}};
    TRON_TRY(dispatch_hv(ds, in, v_dev, partials, fin));
    if (narrow) hipLaunchKernelGGL(k_dense_finish, dim3(1), dim3(kFinishBlock), 0, ds->stream, (int)ds->d, grid, partials, fin);
    TRON_HIP(hipGetLastError());
    return launch_columns(ds, grid, partials, colprod, nullptr, nullptr, fin);
}
