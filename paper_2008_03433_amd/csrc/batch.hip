// Several problems of Section 3 of the paper over one resident dense matrix: the cross-validation setting of
// Section 2.1 (three folds, nested cross-validation inside each), where the problems differ only in the instances
// they train on and in C.  The problems advance in lock-step rounds.  A round is
//   1. one pass over X (k_batch_pass on the vector units, up to eight problems; k_batch_pass_mfma on the fp64 matrix
//      units, up to sixteen) that serves every problem's pending request -- X^T (D (X v)) for a problem inside its CG
//      iteration, or z = X w / loss / D / X^T zhat for one at a trial point (Table 1) -- so that an element of X read
//      from HBM is used by all of them;
//   2. one small kernel (k_batch_advance) that adds up the pass's per-workgroup partial sums and then runs, for every
//      problem, the step of Algorithm 1 / of the truncated CG iteration that was waiting for the product, and posts
//      the problem's next request.
// The trust-region logic runs on the device (device_driver.h).  The host only watches which problems are still running.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <optional>
#include <thread>
#include <type_traits>

#include "dense_tile.h"
#include "device_driver.h"

namespace tron {
namespace {

typedef const uint64_t __attribute__((address_space(4))) *ConstWords;

// ------------------------------------------------------------------ the pass over X
// Work layout as in the single-problem kernels: a wave tile is 64 consecutive rows, a wavefront walks a contiguous
// range of tiles.  Per tile and problem one 64-bit word says which rows concern the problem: its members
// (function/gradient pass, logistic Hessian) or its active set I (L2-SVM Hessian: D_ii = 2 on I).  Rows that concern no
// problem are not read.  The words of the next tile are fetched (scalar loads) while the current one is processed.
// New active-set words are collected in LDS and stored kHeld tiles at a time.
// STREAM: matrices that do not fit the cache come through LDS (TileStream), a tile ahead.  us a function-gradient / Hessian call over 10M x 24: three
// L2-SVMs 373 / 358 loaded, 333 / 312 streamed, six 448 / 358 and 418 / 333, three logistic problems 549 / 415 and 441 / 331; six L2-SVMs
// over 1.4M x 24, which fits, 81 / 65 and 82 / 67.
// What bounds it: instructions and memory in turn, as two wavefronts a SIMD do not cover each other's waits (six L2-SVMs over 1M x 24: vector units
// 45% busy).  So the loop over the problems asks nothing but whether a problem has rows in the tile (see sweep), and the sums over the
// lanes at the end are moves between lanes with one barrier for all problems: pass of 56 / 45 us before, 52 / 38 now.
//   member: [k][tile]     Dbits: [k][slot][tile]     Dval (logistic D): [k][slot][row]
//   partials: [k][column 0..d-1, then the loss sum][workgroup]
// Dbits_in and Dbits_out are the same array: a problem's plane is either read (MODE_HV) or written (MODE_FG) by a pass.
template <int E, int L, int U, bool VEC, int KT, int LOSS, bool STREAM>
__global__ __launch_bounds__(kBlock, 2) void k_batch_pass(int64_t n, int64_t d, const double *__restrict__ X,
                                                       const int8_t *__restrict__ y,
                                                       const BatchCtl *__restrict__ ctl, const uint64_t *__restrict__ member,
                                                       const uint64_t *__restrict__ Dbits_in, uint64_t *Dbits_out,
                                                       double *Dval, int64_t ntiles, double *__restrict__ partials, int /* K: unused here */)
{
    using T = Tile<E, L, U, VEC>;
    static_assert(T::RT == kWave, "one 64-bit word per tile");
    __shared__ double lvec[KT][E * L];
    __shared__ double lcols[STREAM ? 1 : kWavesPerBlock][KT][E * L];
    __shared__ double lds_red[kWavesPerBlock][KT];
    // function/gradient pass only, kept out of the registers: per wavefront and problem the loss sum of every lane's rows
    // and the new active-set words of up to kHeld tiles
    __shared__ double lloss[kWavesPerBlock][KT][kWave];
    __shared__ double lprod[LOSS == TRON_LOSS_LR ? kWavesPerBlock : 1][KT][kWave];   // and their product, see LossSum
    constexpr int kHeld = KT > 4 ? (STREAM ? 16 : 64) : 32;
    __shared__ uint64_t lheld[kWavesPerBlock][KT][LOSS == TRON_LOSS_LR ? 1 : kHeld];
    extern __shared__ __align__(16) double dyn[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int q = lane % L, own = T::own_row(lane);
    int mode[KT], dslot[KT];
    unsigned live = 0, fg = 0, hv = 0;   // problems by what they ask for
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        mode[k] = ctl->mode[k];
        dslot[k] = ctl->dslot[k];
        live |= (unsigned)(mode[k] != MODE_IDLE) << k;
        fg |= (unsigned)(mode[k] == MODE_FG) << k;
        hv |= (unsigned)(mode[k] == MODE_HV) << k;
    }
    if (live == 0) return;
    constexpr bool svm = LOSS == TRON_LOSS_L2SVM;
    // plane of the words that say which rows concern problem k.  The words are the same for all lanes: read through
    // the constant address space they arrive in scalar registers.  (No plane read here is written by this pass.)
    ConstWords words[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        if ((mode[k] == MODE_HV || mode[k] == MODE_DIAG) && svm) words[k] = (ConstWords)(Dbits_in + ((int64_t)k * 2 + dslot[k]) * ntiles);
        else words[k] = (ConstWords)(member + (int64_t)k * ntiles);
    }
    const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t wave_id = (int64_t)blockIdx.x * kWavesPerBlock + wv;
    const int64_t per_wave = (ntiles + nwaves - 1) / nwaves;
    const int64_t first = wave_id * per_wave;
    const int64_t last = (first + per_wave < ntiles) ? first + per_wave : ntiles;
    uint64_t wnext[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k) wnext[k] = (mode[k] != MODE_IDLE && first < last) ? words[k][first] : 0;
    // L2-SVM Hessian: D_ii = 2 on the active set.  The factor is put into v (exact: a power of two), the product
    // then only selects rows.
    for (int i = threadIdx.x; i < KT * E * L; i += kBlock) {
        const int k = i / (E * L), at = i % (E * L), c = T::col(at / E, at % E);   // lane q's entries lie together
        const double scale = (svm && ctl->mode[k] == MODE_HV) ? 2.0 : 1.0;
        lvec[k][at] = (c < d) ? scale * ctl->vec[k][c] : 0.0;
    }
    __syncthreads();
    double acc[KT][E];
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        lloss[wv][k][lane] = 0.0;
        if (!svm) lprod[wv][k][lane] = 0.0;
        if (svm && lane < kHeld) lheld[wv][k][lane] = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[k][e] = 0.0;
    }
    // The pass over the wavefront's tiles.  M: what every problem that is not idle asks for, or kMixed.  Knowing it takes the questions out of
    // the loop over the problems: they were 305 scalar instructions a tile beside 845 vector ones (six problems, 24 columns).
    constexpr int kMixed = -1;
    auto sweep = [&](auto what) __attribute__((always_inline)) {
        constexpr int M = decltype(what)::value;
        const auto mode_of = [&](int k) { return M == kMixed ? mode[k] : M; };
        const bool any_fg = M == kMixed ? fg != 0 : M == MODE_FG;
        // What travels with a tile's rows: its labels, and for the logistic Hessian D of every problem, a lane taking the row it owns.
        TileStream<E, L, U, VEC> stream(STREAM ? dyn : nullptr, d);
        double ynext = 1.0, Dnext[KT];
        auto ask = [&](int64_t tile, const uint64_t (&w)[KT]) {
            uint64_t rows = 0;
#pragma unroll
            for (int k = 0; k < KT; ++k) rows |= w[k];
            stream.ask(X, n, d, tile, tile < last && __popcll(rows) >= kWave / 2);
            const bool mine = tile < last && tile * kWave + own < n;
            ynext = (any_fg && mine) ? (double)y[tile * kWave + own] : 1.0;
            if constexpr (!svm) {
#pragma unroll
                for (int k = 0; k < KT; ++k) {
                    Dnext[k] = 0.0;
                    if ((mode_of(k) == MODE_HV || mode_of(k) == MODE_DIAG) && w[k] != 0 && mine)
                        Dnext[k] = Dval[((int64_t)k * 2 + dslot[k]) * n + tile * kWave + own];   // zero outside the problem's rows
                }
            }
        };
        ask(first, wnext);
        int it = 0;
        for (int64_t tile = first; tile < last; ++tile, ++it) {
            const int slotl = it & (kHeld - 1);
            const int64_t row0 = tile * kWave, ahead = tile + 1 < last ? tile + 1 : tile;
            uint64_t wk[KT], rows = 0;
#pragma unroll
            for (int k = 0; k < KT; ++k) {
                wk[k] = wnext[k];
                rows |= wk[k];
                wnext[k] = (live >> k & 1u) ? words[k][ahead] : 0;
            }
            double x[U][E], Drow[KT];
            if (rows != 0) stream.take(X, n, d, tile, lane, x, rows);
            const double yrow = ynext;
            if constexpr (!svm) {
#pragma unroll
                for (int k = 0; k < KT; ++k) Drow[k] = Dnext[k];
            }
            ask(tile + 1, wnext);
            if (rows != 0) {
                if (M == kMixed && live != (fg | hv)) {   // uniform
#pragma unroll
                    for (int k = 0; k < KT; ++k) {
                        if (mode[k] != MODE_DIAG || wk[k] == 0) continue;   // uniform
                        // sum_i D_i x_ij^2: the row coefficient is D itself, the entries are squared
                        double c[U];
                        T::from_row_owner(svm ? (((wk[k] >> own) & 1u) ? 2.0 : 0.0) : Drow[k], c);
#pragma unroll
                        for (int u = 0; u < U; ++u) {
#pragma unroll
                            for (int e = 0; e < E; ++e) acc[k][e] = fma(c[u] * x[u][e], x[u][e], acc[k][e]);
                        }
                    }
                }
                // The vectors are read from LDS again for every tile: hoisted out of the loop they would take KT * E
                // registers per lane (the empty statement hides the loop invariance from the compiler).  Each is asked for a problem
                // ahead where there are registers for it.
                int qoff = q * E;
                asm volatile("" : "+v"(qoff));
                constexpr bool kAhead = KT * E <= (svm ? 56 : 32);
                double vnext[E];
#pragma unroll
                for (int e = 0; kAhead && e < E; ++e) vnext[e] = lvec[0][qoff + e];
#pragma unroll
                for (int k = 0; k < KT; ++k) {
                    double vk[E], c[U];
#pragma unroll
                    for (int e = 0; kAhead && e < E; ++e) {
                        vk[e] = vnext[e];
                        if (k + 1 < KT) vnext[e] = lvec[k + 1][qoff + e];
                    }
                    if (wk[k] == 0 || mode_of(k) == MODE_DIAG) continue;   // uniform (no bit: nothing asked for, or no row)
#pragma unroll
                    for (int e = 0; !kAhead && e < E; ++e) vk[e] = lvec[k][qoff + e];
                    const bool mine = (wk[k] >> own) & 1u;
                    const double z = T::row_sum(x, vk, lane);
                    double coef;
                    if (mode_of(k) == MODE_HV) {
                        coef = svm ? (mine ? z : 0.0) : Drow[k] * z;   // a1 = D (X v) in the row's owner
                    } else {
                        // the per-row terms of Table 1 run once per row
                        LossTerm alpha;
                        double zhat, Di;
                        loss_terms_dev<LOSS>(z, yrow, alpha, zhat, Di);
                        if (!mine) { alpha = LossTerm{0.0, 0.0}; zhat = 0.0; Di = 0.0; }
                        if constexpr (svm) {
                            lds_add(&lloss[wv][k][lane], alpha.lin);
                            const uint64_t nb = __ballot(Di != 0.0);
                            if (lane == 0) lheld[wv][k][slotl] = nb;   // in the order of the lanes
                        } else {
                            LossSum<LOSS> losses{lloss[wv][k][lane], lprod[wv][k][lane]};
                            losses.add(alpha);
                            lloss[wv][k][lane] = losses.lin;
                            lprod[wv][k][lane] = losses.p;
                            if (mine) Dval[((int64_t)k * 2 + dslot[k]) * n + row0 + own] = Di;
                        }
                        coef = zhat;
                    }
                    T::from_row_owner(coef, c);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
#pragma unroll
                        for (int e = 0; e < E; ++e) acc[k][e] = fma(c[u], x[u][e], acc[k][e]);
                    }
                }
            }
            if constexpr (!svm) {
                // by the number of the tile, whichever problems have rows in it: none of them adds more than once a tile
                if (any_fg && (it & (LossSum<LOSS>::kAdds - 1)) == LossSum<LOSS>::kAdds - 1) {
#pragma unroll
                    for (int k = 0; k < KT; ++k) {
                        LossSum<LOSS> losses{lloss[wv][k][lane], lprod[wv][k][lane]};
                        losses.scale();
                        lloss[wv][k][lane] = losses.lin;
                        lprod[wv][k][lane] = losses.p;
                    }
                }
            }
            if (svm && any_fg && (slotl == kHeld - 1 || tile + 1 == last)) {
                // lane i takes the word of tile (tile - slotl + i): consecutive 8-byte words per problem
#pragma unroll
                for (int k = 0; k < KT; ++k) {
                    if ((fg >> k & 1u) && lane <= slotl)
                        Dbits_out[((int64_t)k * 2 + dslot[k]) * ntiles + (tile - slotl) + lane] = T::rows_of_ballot(lheld[wv][k][lane]);
                    if (lane < kHeld) lheld[wv][k][lane] = 0;
                }
            }
        }
    };
    if (live == hv) sweep(std::integral_constant<int, MODE_HV>{});
    else if (live == fg) sweep(std::integral_constant<int, MODE_FG>{});
    else sweep(std::integral_constant<int, kMixed>{});
    // columns and loss sums over the wavefronts, in order
    double *const cols_w = STREAM ? dyn + wv * (kWave * d) : &lcols[STREAM ? 0 : wv][0][0];   // (the rows in the wavefront's part have been read)
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        if (!(live >> k & 1u)) continue;   // uniform
        T::sum_columns(acc[k]);
        if (lane < L) {
#pragma unroll
            for (int e = 0; e < E; ++e) cols_w[k * (E * L) + T::col(lane, e)] = acc[k][e];
        }
        if (fg >> k & 1u) {
            const double ls = wave_sum(LossSum<LOSS>{lloss[wv][k][lane], svm ? 0.0 : lprod[svm ? 0 : wv][k][lane]}.value());
            if (lane == 0) lds_red[wv][k] = ls;
        } else if (lane == 0) lds_red[wv][k] = 0.0;
    }
    __syncthreads();
    const int cols = (int)d + 1;
    for (int i = threadIdx.x; i < KT * cols; i += kBlock) {
        const int k = i / cols, c = i - k * cols;
        if (!(live >> k & 1u)) continue;
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w)
            s += c == (int)d ? lds_red[w][k] : (STREAM ? dyn[w * (kWave * d) + k * (E * L) + c] : lcols[STREAM ? 0 : w][k][c]);
        partials[(int64_t)i * gridDim.x + blockIdx.x] = s;
    }
}

// ------------------------------------------------------------------ the pass over X on the matrix units
// With several problems the pass is two skinny matrix products per tile of 64 rows: Z = X V (64 x d by d x K) and
// G += X^T C (d x 64 by 64 x K), C = the row coefficients formed from Z.  This kernel runs them as fp64 matrix
// instructions (16 x 16 x 4: A 16 x 4, B 4 x 16, result 16 x 16; lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and, in
// its result register v, the element [4 v + l / 16][l % 16]) with the problems as the 16 result columns:
//   * a wavefront copies its tile of X into LDS exactly as it lies in memory (16-byte pieces, the loads of the next tile
//     in flight during the work on the current one; rows that concern no problem are not read);
//   * Z: per 16 rows and 4 columns of X one instruction, A read from LDS, B = V kept in registers;
//   * lane (g = l / 16, p = l % 16) then holds Z of problem p at rows 4 v + g of every 16-row group, and C is formed where
//     Z lies.  Hessian rounds: the L2-SVM selects by the bit of the active-set word (factor 2 folded into V), the
//     logistic loss multiplies by D, which each lane loads for its own elements (four consecutive rows of a problem
//     per instruction and group of lanes; the four instructions of a 16-row step use up whole lines).  Function/gradient rounds of the
//     L2-SVM: the lane evaluates the loss terms of its own sixteen (row, problem) elements per tile (the same
//     per-element function as k_batch_pass; labels and membership come as bits of two 64-bit words per tile), keeps one
//     loss sum -- its problem's -- and its rows' bits of the new active-set word, which the four lanes of a problem put
//     together once per tile.  The logistic terms (an exponential, a logarithm and a division each) cost more than
//     everything else in the pass, so they are evaluated once per row and problem that asks -- not for the sixteen
//     result columns: Z goes through an LDS exchange area to a row-per-lane layout, where the new D is stored as
//     64 consecutive rows of a problem, and zhat comes back the same way;
//   * G: the result rows are the columns of X (two instructions for d > 16); the four rows 4 v + g, g = 0..3, that the
//     lanes hold in register v are the summation index, so C is used where it lies.  A = X[row][column] read from LDS
//     along a row: conflict-free.  Problems asking for the Hessian diagonal use the same instructions with A squared and
//     C = D.
// What bounds it: a Hessian round 12 logistic problems x 24 columns memory (20M rows: 3.84 GB of X and 1.92 GB of D in 1.0 ms), now that a tile takes
// 195 vector instructions, 56 of them matrix ones, and 190 scalar ones; it took 503 and 450, and 1.05 ms, with the problems' modes looked up for each
// element, 32 lane reads for the union of the words, selects for rows and places that are all there, and addresses formed a lane at
// a time.  A function-gradient round instructions: 1180 vector ones a tile (1420), half of them loss terms, 1.75 ms (1.81).  us a
// call of 12 problems over 4M rows, before / now, Hessian: 24 columns logistic 246 / 223, L2-SVM 189 / 182; 17 columns 240 / 217, 225 / 189; function-gradient
// 10 columns 324 / 300, 180 / 155; 30 columns 426 / 429, 277 / 256.
// Results go to the same partials array, in the same layout, as k_batch_pass writes: the steps after the pass do not
// know which kernel ran.  Sums are formed in a fixed order (the instruction's, then tiles in order, wavefronts 0..3).
typedef double mfma4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void wave_lds_fence()
{
    // LDS operations of one wavefront complete in the order issued; this keeps the compiler from reordering them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// the 64-bit value of lane `src` (per-lane index)
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int src)
{
    const int lo = __builtin_amdgcn_ds_bpermute(src * 4, (int)(uint32_t)v);
    const int hi = __builtin_amdgcn_ds_bpermute(src * 4, (int)(uint32_t)(v >> 32));
    return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

// doubles of LDS per wavefront: a unit of RT rows of X (rows padded to at most dmax + 2 doubles, 16 doubles of slack) and,
// where logistic function / gradient requests are served (kex = K, otherwise 0), the exchange area: kex rows of RT + 1
// doubles for Z and zhat by problem and row
__host__ __device__ constexpr int mfma_wave_doubles(int dmax, int kex, int rt) { return rt * (dmax + 2) + 16 + ((kex * (rt + 1) + 1) & ~1); }

__device__ __align__(16) double kNoRow[2] = {0.0, 0.0};   // what is read instead of rows that concern no problem

// RT = rows of X a wavefront keeps in LDS at a time: a whole 64-row tile, or half of one (smaller LDS footprint and
// fewer registers for the loads in flight, so more wavefronts per SIMD to cover the dependent chains of matrix
// instructions; the row-per-lane steps then serve 64 / RT problems side by side).
// FG = false: a pass in which no problem asks for function and gradient (the host knows the modes of the round).  The
// per-element loss terms, the labels, the loss sums and the new active-set words are compiled out: fewer registers, so
// more wavefronts per SIMD.
template <bool VEC, int DMAX, int KT, int LOSS, int RT, bool FG>
__global__ __launch_bounds__(kBlock, FG ? 2 : 3) void k_batch_pass_mfma(int64_t n, int64_t d, const double *__restrict__ X,
                                                            const int8_t *__restrict__ y,
                                                            const BatchCtl *__restrict__ ctl, const uint64_t *__restrict__ member,
                                                            const uint64_t *__restrict__ Dbits_in, uint64_t *Dbits_out,
                                                            double *Dval, int64_t ntiles, double *__restrict__ partials, int K)
{
    static_assert(KT <= 16 && KT <= kBatchMax, "one result column per problem");
    static_assert(RT == 32 || RT == 64, "a tile or half a tile");
    constexpr bool svm = LOSS == TRON_LOSS_L2SVM;
    static_assert(DMAX % 4 == 0 && DMAX <= kVecPad, "d <= DMAX, in steps of the instruction's four columns");
    constexpr int PW = VEC ? 2 : 1;                 // doubles per piece
    constexpr int NH = kWave / RT;                  // units per tile
    constexpr int NS = RT / 16;                     // groups of 16 rows per unit
    constexpr int NP = RT * DMAX / PW / kWave;      // pieces per lane and unit at most (a unit is RT d doubles)
    constexpr int PP = kWave / RT;                  // problems side by side in the row-per-lane layout
    static_assert(RT * DMAX / PW % kWave == 0 && KT % PP == 0, "whole pieces per lane; whole groups of problems");
    constexpr int kExRow = RT + 1;                  // doubles per problem in the exchange area (padded against bank conflicts)
    constexpr bool kHasEx = FG && !svm;             // logistic function / gradient requests go through the exchange area
    extern __shared__ double dyn[];
    __shared__ double lds_red[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int D = (int)d;
    int mode[KT], dslot[KT];
    unsigned live = 0, fg = 0, hv = 0;   // problems by what they ask for
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        mode[k] = ctl->mode[k];
        dslot[k] = ctl->dslot[k];
        live |= (unsigned)(mode[k] != MODE_IDLE) << k;
        fg |= (unsigned)(mode[k] == MODE_FG) << k;
        hv |= (unsigned)(mode[k] == MODE_HV) << k;
    }
    if (live == 0) return;
    // The unit in LDS: row r at r S, S = the first length >= d whose rows start in different banks for 16 consecutive rows
    // (16-byte pieces: S = 2 mod 4; 8-byte pieces: S odd).  Every lane copies NP pieces per unit; those past the unit
    // (d < DMAX) are zeros and land in the slack behind it.
    constexpr int xs_len = RT * (DMAX + 2) + 16;
    const int S = VEC ? D + ((6 - D % 4) % 4) : (D | 1);
    const int kex = kHasEx ? K : 0;
    double *Xs = dyn + (size_t)wv * mfma_wave_doubles(DMAX, kex, RT);
    double *Ex = Xs + xs_len;                                    // [problem][row of the unit]: Z, then zhat
    for (int i = lane; i < mfma_wave_doubles(DMAX, kex, RT); i += kWave) Xs[i] = 0.0;
    // this lane in the matrix layouts: g = summation index / row block, p = problem (result column) or row / column of X
    const int p = lane & 15, g = lane >> 4;
    const bool pk = p < K;   // K <= KT
    const int modeM = pk ? ctl->mode[pk ? p : 0] : MODE_IDLE;
    const int dslotM = pk ? ctl->dslot[pk ? p : 0] : 0;
    const bool exM = !svm && (modeM == MODE_HV || modeM == MODE_DIAG);   // this lane's problem reads its D
    const int rowl = lane & (RT - 1), sub = lane / RT;   // row-per-lane layout: row of the unit, problem of a group of PP
    // logistic D of this lane's problem in the slot it reads; lanes without such a problem stay at the start of the array
    const double *const DvalM = (!svm && pk) ? Dval + ((int64_t)p * 2 + dslotM) * n : Dval;
    // where every problem is in its Hessian product, the other lanes read along with the first problem (their result columns nobody reads)
    const int pA = __ffs(live) - 1;
    const double *const DvalH = (!svm && modeM == MODE_IDLE) ? Dval + ((int64_t)pA * 2 + ctl->dslot[pA]) * n : DvalM;
    double Vop[DMAX / 4];
#pragma unroll
    for (int kk = 0; kk < DMAX / 4; ++kk) {
        const int f = 4 * kk + g;
        const bool use = f < D && (modeM == MODE_HV || (FG && modeM == MODE_FG));
        const double scale = (svm && modeM == MODE_HV) ? 2.0 : 1.0;
        Vop[kk] = use ? scale * ctl->vec[pk ? p : 0][f] : 0.0;
    }
    // lane k < KT fetches the word of problem k: its active set (L2-SVM Hessian / diagonal) or its members
    const uint64_t *plane = nullptr;
    if (lane < KT) {
        const int m = ctl->mode[lane < KT ? lane : 0];
        if ((m == MODE_HV || m == MODE_DIAG) && svm) plane = Dbits_in + ((int64_t)lane * 2 + ctl->dslot[lane < KT ? lane : 0]) * ntiles;
        else if (m != MODE_IDLE) plane = member + (int64_t)lane * ntiles;
    }
    const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t wave_id = (int64_t)blockIdx.x * kWavesPerBlock + wv;
    const int64_t per_wave = (ntiles + nwaves - 1) / nwaves;
    const int64_t first = wave_id * per_wave;
    const int64_t last = (first + per_wave < ntiles) ? first + per_wave : ntiles;
    const uint64_t inv_d = (0x100000000ull + (uint64_t)D - 1) / (uint64_t)D;   // row of element e < 2048: (e inv_d) >> 32 (2^32 itself for d = 1)
    // per piece of this lane, fixed for the whole pass: where it goes in LDS
    uint32_t plds[NP];
#pragma unroll
    for (int it = 0; it < NP; ++it) {
        const uint32_t e = (uint32_t)(it * kWave + lane) * PW;
        const uint32_t row = (uint32_t)(((uint64_t)e * inv_d) >> 32);
        plds[it] = row < (uint32_t)RT ? row * (uint32_t)S + (e - row * (uint32_t)D) : (uint32_t)(xs_len - 2);
    }

    const int pieces = RT * D / PW;   // of a unit
    const bool once = !FG && read_once(n, d);   // (a round with loss terms is not bound by memory)
    double xr[NP][PW];
#pragma unroll
    for (int it = 0; it < NP; ++it)
#pragma unroll
        for (int e = 0; e < PW; ++e) xr[it][e] = 0.0;
    double lossM = 0.0;   // L2-SVM: loss terms of this lane's rows of its problem
    LossSum<LOSS> lossK[KT / PP];   // logistic: losses of this lane's row, by problem (PP k + sub)
    int adds = 0;
    uint64_t nbM = 0;     // this lane's rows' bits of its problem's new active-set word for the current tile
    mfma4 G1 = {0.0, 0.0, 0.0, 0.0}, G2 = {0.0, 0.0, 0.0, 0.0};

    // the rows of unit h of a tile that concern some problem
    auto unit_rows = [&](uint64_t rows, int h) -> uint64_t { return RT == kWave ? rows : ((rows >> (RT * h)) & 0xffffffffull); };
    // Loads of a unit into xr, then xr into LDS.  No load sits behind a branch on a per-lane condition (the compiler would
    // wait for every load in flight where such paths join): for a piece of a row that concerns no problem, or past the end,
    // zeros are fetched (kNoRow: one cached line for all of them) and copied like the others.  What lies in such a row counts for nothing.
    auto fetch = [&](int64_t tile, int h, uint64_t urows) __attribute__((always_inline)) {
        const int64_t row0 = tile * kWave + RT * h;
        const double *base = X + row0 * d;
        const bool full = urows == (RT == kWave ? ~0ull : 0xffffffffull) && row0 + RT <= n;
        auto load = [&](int it, const double *src) __attribute__((always_inline)) {
            if constexpr (VEC) {
                const double2 t = *reinterpret_cast<const double2 *>(src);
                xr[it][0] = t.x;
                xr[it][1] = t.y;
            } else {
                xr[it][0] = *src;
            }
        };
        if (full) {   // no per-row questions; the same address in every lane but for its own place.  Pieces past the unit keep what they hold.
            if (once) {   // (see read_once)
                auto at = (const __attribute__((address_space(1))) double *)(base + lane * PW);
                asm volatile("" : "+v"(at));   // (otherwise the compiler makes one ordinary load of these and those below)
#pragma unroll
                for (int it = 0; it < NP; ++it) {
                    if (it >= pieces / kWave) {
                        if (it * kWave < pieces) load(it, it * kWave + lane < pieces ? base + it * kWave * PW + lane * PW : kNoRow);
                    } else if constexpr (VEC) {
                        const v2d t = __builtin_nontemporal_load((const __attribute__((address_space(1))) v2d *)(at + it * kWave * PW));
                        xr[it][0] = t.x;
                        xr[it][1] = t.y;
                    } else xr[it][0] = __builtin_nontemporal_load(at + it * kWave * PW);
                }
                return;
            }
#pragma unroll
            for (int it = 0; it < NP; ++it) {
                if (it < pieces / kWave) load(it, base + it * kWave * PW + lane * PW);   // uniform
                else if (it * kWave < pieces) load(it, it * kWave + lane < pieces ? base + it * kWave * PW + lane * PW : kNoRow);
            }
            return;
        }
#pragma unroll
        for (int it = 0; it < NP; ++it) {
            uint32_t at = (uint32_t)lane;
            asm volatile("" : "+v"(at));   // (not to be kept in registers for all units)
            const uint32_t e = (it * kWave + at) * PW, row = (uint32_t)(((uint64_t)e * inv_d) >> 32);
            const bool take = row < (uint32_t)RT && ((urows >> (row & (RT - 1))) & 1u) && row0 + row < n;
            load(it, take ? base + e : kNoRow);
        }
    };
    auto to_lds = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < NP; ++it) {
            if constexpr (VEC) *reinterpret_cast<double2 *>(Xs + plds[it]) = make_double2(xr[it][0], xr[it][1]);
            else Xs[plds[it]] = xr[it][0];
        }
    };
    const uint64_t *plane_c = plane ? plane : member;   // a valid address for the lanes that fetch no word
    // raw loads (clamped addresses); what they are worth is decided where they are used, so that nothing waits for them early
    auto word_raw = [&](int64_t tile) { return plane_c[tile < last ? tile : last - 1]; };
    auto word_ok = [&](int64_t tile) { return plane != nullptr && tile < last; };
    auto label_raw = [&](int64_t tile, int h) {
        const int64_t i = tile * kWave + RT * h + rowl;
        return (int)y[i < n ? i : n - 1];   // rows past n belong to no problem: their label is never used
    };
    // a value that is the same within each group of RT lanes: x[sub] of PP values that are the same for every lane
    auto by_sub_i = [&](const int *x) { return (PP == 1 || sub == 0) ? x[0] : x[PP - 1]; };
    auto by_sub_u = [&](const uint64_t *x) { return (PP == 1 || sub == 0) ? x[0] : x[PP - 1]; };
    static_assert(PP <= 2, "by_sub picks between two");

    // words of the current tile (w0), the next (w1) and the one after (loaded in the loop); their scalar copies
    uint64_t w0 = 0, w1 = 0;
    if (first < last) {   // the same for the whole wavefront
        w0 = word_ok(first) ? word_raw(first) : 0ull;
        w1 = word_ok(first + 1) ? word_raw(first + 1) : 0ull;
    }
    // Scalar copies of the problems' words (where a row's terms are formed problem by problem), and the rows that concern any of them
    uint64_t wk[kHasEx ? KT : 1];
    auto scalar_words = [&](uint64_t w, uint64_t (&each)[kHasEx ? KT : 1]) __attribute__((always_inline)) -> uint64_t {
        uint64_t rows = 0;
        if constexpr (kHasEx) {
#pragma unroll
            for (int k = 0; k < KT; ++k) {
                each[k] = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(w >> 32), k) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)w, k);
                rows |= each[k];
            }
        } else {   // over the first sixteen lanes
            int lo = (int)(uint32_t)w, hi = (int)(uint32_t)(w >> 32);
            auto fold = [](int v) {
                v |= __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true);   // row_ror:8, 4, 2, 1
                v |= __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, true);
                v |= __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, true);
                return v | __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, true);
            };
            rows = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(fold(hi)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane(fold(lo));
        }
        return rows;
    };
    uint64_t rows_cur = scalar_words(w0, wk);
    // The wavefront's tiles.  M: what every problem that is not idle asks for, or kMixed.
    constexpr int kMixed = -1;
    auto sweep = [&](auto what) __attribute__((always_inline)) {
        constexpr int M = decltype(what)::value;
        const bool any_fg = FG && (M == kMixed ? fg != 0 : M == MODE_FG), any_hv = M == kMixed ? hv != 0 : M == MODE_HV;
        const bool any_diag = M == kMixed && live != (fg | hv), any_mul = M != kMixed || (FG ? (fg | hv) : hv) != 0;
        const bool any_exd = !svm && (M == kMixed ? live != fg : M == MODE_HV);
        const auto mode_of = [&](int k) { return M == kMixed ? mode[k] : (live >> k & 1u) ? M : MODE_IDLE; };
        // a lane whose problem is idle, or that has none, forms something finite or not that nobody reads
        const int modeL = M == kMixed ? modeM : M;
        int ycur = 1;   // the labels travel with the unit: asked for with its loads, first touched after they have all arrived
        if (first < last && unit_rows(rows_cur, 0) != 0) {
            if (any_fg) ycur = label_raw(first, 0);
            fetch(first, 0, unit_rows(rows_cur, 0));
        }
        for (int64_t tile = first; tile < last; ++tile) {
            const uint64_t w2 = word_raw(tile + 2);
            uint64_t wkn[kHasEx ? KT : 1];
            const uint64_t rows_next = scalar_words(w1, wkn);
            // the word of this lane's problem
            uint64_t wordM = 0;
            if (svm || any_fg) wordM = lane_value(w0, p);
#pragma unroll 1
            for (int h = 0; h < NH; ++h) {
                const uint64_t urows = unit_rows(rows_cur, h);
                if (urows != 0) to_lds();
                // the loads of the unit after this one
                int ynext = 1;
                {
                    const bool same_tile = h + 1 < NH;
                    const int64_t nt = same_tile ? tile : tile + 1;
                    const int nh = same_tile ? h + 1 : 0;
                    const uint64_t nrows = unit_rows(same_tile ? rows_cur : rows_next, nh);
                    if (nt < last && nrows != 0) {
                        if (any_fg) ynext = label_raw(nt, nh);
                        fetch(nt, nh, nrows);
                    }
                }
                if (urows != 0) {
                    wave_lds_fence();
                    // Z = X V for rows 16 s .. 16 s + 15 of the unit
                    auto z_of = [&](int s) {
                        mfma4 z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                        for (int kk = 0; kk < DMAX / 4; ++kk) {   // columns past d: V is zero there and what A reads is finite
                            const double a = Xs[(16 * s + p) * S + 4 * kk + g];
                            z = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Vop[kk], z, 0, 0, 0);
                        }
                        return z;
                    };
                    if (kHasEx && any_fg) {
                        // logistic function / gradient requests: Z to the row-per-lane layout, the terms once per row and
                        // problem that asks (D stored from there), zhat back
#pragma unroll 1
                        for (int s = 0; s < NS; ++s) {
                            const mfma4 z = z_of(s);
                            if (pk && modeL == MODE_FG) {
#pragma unroll
                                for (int v = 0; v < 4; ++v) Ex[p * kExRow + 16 * s + 4 * v + g] = z[v];
                            }
                        }
                        wave_lds_fence();
                        const double yrow = (double)ycur;
#pragma unroll
                        for (int k = 0; k < KT; k += PP) {
                            bool some = false;
                            int mk[PP], dk[PP];
                            uint64_t wq[PP];
#pragma unroll
                            for (int j = 0; j < PP; ++j) {
                                mk[j] = mode_of(k + j);
                                dk[j] = dslot[k + j];
                                wq[j] = wk[k + j];
                                some |= mk[j] == MODE_FG;
                            }
                            if (!some) continue;   // uniform
                            const int kk = k + sub;
                            const bool act = by_sub_i(mk) == MODE_FG && kk < K;
                            const double z = Ex[(kk < K ? kk : 0) * kExRow + rowl];
                            const bool mine = act && ((by_sub_u(wq) >> (RT * h + rowl)) & 1u);
                            LossTerm alpha;
                            double zhat, Di;
                            loss_terms_dev<LOSS>(z, yrow, alpha, zhat, Di);
                            if (!mine) { alpha = LossTerm{0.0, 0.0}; zhat = 0.0; Di = 0.0; }
                            lossK[k / PP].add(alpha);
                            if (mine) Dval[((int64_t)kk * 2 + by_sub_i(dk)) * n + tile * kWave + RT * h + rowl] = Di;
                            if (act) Ex[kk * kExRow + rowl] = zhat;
                        }
                        if ((++adds & (LossSum<LOSS>::kAdds - 1)) == 0) {
#pragma unroll
                            for (int k = 0; k < KT / PP; ++k) lossK[k].scale();
                        }
                        wave_lds_fence();
                    }
                    // labels of the unit's rows as a word (the same in every lane)
                    const uint64_t yword = (svm && any_fg) ? __ballot(ycur > 0) : 0ull;
                    // G += X^T C, 16 rows at a time
#pragma unroll 1
                    for (int s = 0; s < NS; ++s) {
                        // logistic D of the lane's four elements, asked for before the products that form Z (zero outside the
                        // problem's rows: never written there); no load sits behind a per-lane branch
                        double ev[4] = {0.0, 0.0, 0.0, 0.0};
                        bool evok[4] = {false, false, false, false};
                        if (M == MODE_HV && any_exd && tile * kWave + kWave <= n) {   // uniform
                            const double *const at = DvalH + (tile * kWave + RT * h + 16 * s + g);
#pragma unroll
                            for (int v = 0; v < 4; ++v) ev[v] = at[4 * v];
                        } else if (any_exd) {   // uniform
                            const int64_t r0 = tile * kWave + RT * h + 16 * s + g;
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                evok[v] = exM && r0 + 4 * v < n;
                                ev[v] = *(evok[v] ? DvalM + r0 + 4 * v : Dval);
                                if (M == MODE_HV && !evok[v]) ev[v] = 0.0;   // rows past n: what lies in LDS in their place is not theirs
                            }
                        }
                        mfma4 z = {0.0, 0.0, 0.0, 0.0};
                        if (any_hv || (svm && any_fg)) z = z_of(s);
                        // every LDS read of the 16 rows first (none behind a per-lane condition), then the selects and the products.
                        // Columns of X past d give result rows that nobody reads: A is used as it lies in LDS.
                        double a1v[4], a2v[4], ex[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int r = 16 * s + 4 * v + g;
                            ex[v] = kHasEx ? Ex[(pk ? p : 0) * kExRow + r] : 0.0;   // zhat of a logistic function / gradient request
                            a1v[v] = Xs[r * S + p];
                            a2v[v] = (DMAX > 16) ? Xs[r * S + 16 + p] : 0.0;
                        }
                        const uint32_t bits = (uint32_t)(wordM >> (RT * h + 16 * s + g));   // bit 4 v: row 16 s + 4 v + g of the unit
                        const uint32_t ybits = (uint32_t)(yword >> (16 * s + g));            // the same rows' labels
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const double e = M == MODE_HV || evok[v] ? ev[v] : 0.0;
                            const bool bit = (bits >> (4 * v)) & 1u;
                            double cfg = 0.0;   // zhat of a function / gradient request
                            if (kHasEx) cfg = (modeL == MODE_FG) ? ex[v] : 0.0;
                            if (svm && any_fg) {   // uniform
                                const double yv = ((ybits >> (4 * v)) & 1u) ? 1.0 : -1.0;
                                double alpha, zhat, Di;   // L2-SVM only
                                loss_terms_dev<LOSS>(z[v], yv, alpha, zhat, Di);
                                const bool mine = modeL == MODE_FG && bit;   // a row of this lane's problem (rows past n have no bit)
                                lossM += mine ? alpha : 0.0;
                                cfg = mine ? zhat : 0.0;
                                const int rt = RT * h + 16 * s + 4 * v + g;   // the row in its tile
                                nbM |= (uint64_t)(mine && Di != 0.0) << rt;
                            }
                            double c;
                            if (svm) c = (modeL == MODE_HV) ? (bit ? z[v] : 0.0) : cfg;
                            else c = (modeL == MODE_HV) ? e * z[v] : cfg;
                            if (any_mul) {
                                G1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1v[v], c, G1, 0, 0, 0);
                                if (DMAX > 16) G2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a2v[v], c, G2, 0, 0, 0);
                            }
                            if (any_diag) {
                                double cd;
                                if (svm) cd = (modeM == MODE_DIAG && bit) ? 2.0 : 0.0;
                                else cd = (modeM == MODE_DIAG) ? e : 0.0;
                                // a square that is too large for a number counts as the largest one: infinity times the zero of a problem
                                // that the row does not concern would be none
                                G1 = __builtin_amdgcn_mfma_f64_16x16x4f64(fmin(a1v[v] * a1v[v], __DBL_MAX__), cd, G1, 0, 0, 0);
                                if (DMAX > 16) G2 = __builtin_amdgcn_mfma_f64_16x16x4f64(fmin(a2v[v] * a2v[v], __DBL_MAX__), cd, G2, 0, 0, 0);
                            }
                        }
                    }
                    wave_lds_fence();   // the next unit is written over this one
                }
                asm volatile("" : "+v"(ynext));   // nothing of the next unit's loads is touched before this point
                ycur = ynext;
            }
            if (svm && any_fg) {
                // the four lanes of a problem hold disjoint rows' bits of its new word; a tile without rows still gets its zero
                uint64_t word = nbM | lane_value(nbM, lane ^ 16);
                word |= lane_value(word, lane ^ 32);
                if (g == 0 && modeM == MODE_FG) Dbits_out[((int64_t)p * 2 + dslotM) * ntiles + tile] = word;
                nbM = 0;
            }
            w0 = w1;
            w1 = word_ok(tile + 2) ? w2 : 0ull;
            rows_cur = rows_next;
#pragma unroll
            for (int k = 0; k < (kHasEx ? KT : 1); ++k) wk[k] = wkn[k];
        }
    };
    if (!FG && live == hv) sweep(std::integral_constant<int, MODE_HV>{});
    else if (FG && live == fg) sweep(std::integral_constant<int, FG ? MODE_FG : kMixed>{});
    else sweep(std::integral_constant<int, kMixed>{});
    // wavefronts 0..3 added in order; result register v of lane (g, p) is column 4 v + g (G1) / 16 + 4 v + g (G2) of problem p
    __syncthreads();
    double *Gs = dyn;   // [wavefront][column 0..31][problem 0..15]
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        Gs[((wv * 32) + 4 * v + g) * 16 + p] = G1[v];
        Gs[((wv * 32) + 16 + 4 * v + g) * 16 + p] = G2[v];
    }
    __syncthreads();
    const int64_t cols = d + 1;
    for (int i = threadIdx.x; i < KT * D; i += kBlock) {
        const int k = i / D, col = i % D;
        if (ctl->mode[k] == MODE_IDLE) continue;
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) t += Gs[((w * 32) + col) * 16 + k];
        partials[((int64_t)k * cols + col) * gridDim.x + blockIdx.x] = t;
    }
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        if (mode[k] == MODE_IDLE) continue;   // uniform over the workgroup
        const double ls = FG ? block_sum(svm ? (p == k ? lossM : 0.0) : (sub == k % PP ? lossK[k / PP].value() : 0.0), lds_red) : 0.0;
        if (threadIdx.x == 0) partials[((int64_t)k * cols + d) * gridDim.x + blockIdx.x] = ls;
    }
}

// ------------------------------------------------------------------ membership words
// planes[k][tile] bit i = bit k of member[tile*64 + i]; rows past n give zero bits.  bad[0] is set when a word has a bit at or above K.
__global__ __launch_bounds__(kBlock) void k_member_planes(int64_t n, int K, const uint32_t *__restrict__ member,
                                                          int64_t ntiles, uint64_t *__restrict__ planes, int *bad)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t tile = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave; tile < ntiles; tile += nwaves) {
        const int64_t row = tile * kWave + lane;
        const uint32_t m = (row < n) ? member[row] : 0u;
        if ((m >> K) != 0u) bad[0] = 1;   // K <= 16
        for (int k = 0; k < K; ++k) {
            const uint64_t b = __ballot((m >> k) & 1u);
            if (lane == 0) planes[(int64_t)k * ntiles + tile] = b;
        }
    }
}

constexpr int kAdvanceBlock = 1024;

// One workgroup per problem.  All sixteen wavefronts add up the pass's partial sums (fixed order); the first one then runs
// the step that was waiting for them.  A wavefront's loads are asked for together, eight of each of its columns (two with d = 24,
// three at most): latency is all there is to it.  One load after the other it took 9.1 us for 512 workgroups of six problems, 17 for 1024 of twelve.
__global__ __launch_bounds__(kAdvanceBlock) void k_batch_advance(int64_t d, int grid, const double *__restrict__ partials,
                                                          BatchCtl *ctl, ProbState *st, SolveParams P,
                                                          tron_trace_rec *trace, BatchHost *host, int64_t stamp)
{
    const int k = blockIdx.x;
    const int mode = ctl->mode[k];
    __shared__ double cs[kVecPad + 1];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    if (mode != MODE_IDLE) {   // uniform
        constexpr int kWaves = kAdvanceBlock / kWave, kColumns = kVecPad / kWaves + 1, kAtOnce = 8;
        const double *p = partials + ((int64_t)k * (d + 1) + wv) * grid;
        double s[kColumns];
#pragma unroll
        for (int j = 0; j < kColumns; ++j) s[j] = 0.0;
        for (int b0 = lane; b0 < grid; b0 += kAtOnce * kWave) {
            double v[kColumns][kAtOnce];
#pragma unroll
            for (int j = 0; j < kColumns; ++j)
#pragma unroll
                for (int i = 0; i < kAtOnce; ++i) {
                    const int b = b0 + i * kWave;
                    v[j][i] = (wv + j * kWaves <= d && b < grid) ? p[(int64_t)j * kWaves * grid + b] : 0.0;
                }
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i)
#pragma unroll
                for (int j = 0; j < kColumns; ++j) s[j] += v[j][i];
        }
#pragma unroll
        for (int j = 0; j < kColumns; ++j) {
            const double t = wave_sum(s[j]);
            if (lane == 0 && wv + j * kWaves <= d) cs[wv + j * kWaves] = t;
        }
        __syncthreads();
    }
    if (wv == 0) advance_problem(k, mode, d, lane < d ? cs[lane] : 0.0, cs[d], ctl, st, P, trace, host, stamp);
}

__global__ __launch_bounds__(kWave) void k_batch_begin(int what, int64_t d, const double *__restrict__ IN, BatchC Cs, BatchCtl *ctl, ProbState *st)
{
    begin_problem(blockIdx.x, what, d, IN, Cs.v[blockIdx.x], ctl, st);
}

// ------------------------------------------------------------------ kernel choice
using PassFn = void (*)(int64_t, int64_t, const double *, const int8_t *, const BatchCtl *, const uint64_t *,
                        const uint64_t *, uint64_t *, double *, int64_t, double *, int);

struct PassPair { PassFn fn[2]; };   // by loss

template <int E, int L, int KT, bool STREAM>
PassPair pass_for(bool vec)
{
    constexpr int U = pick_U(E, L);
    constexpr bool S = STREAM && tiles_stream(L);
    if constexpr (S && KT == 8) {   // (the logistic kernel has no room for the tiles)
        if constexpr (E % 2 == 0) {
            if (vec) return {{nullptr, k_batch_pass<E, L, U, true, KT, TRON_LOSS_L2SVM, S>}};
        }
        return {{nullptr, k_batch_pass<E, L, U, false, KT, TRON_LOSS_L2SVM, S>}};
    } else {
    if constexpr (E % 2 == 0) {
        if (vec) return {{k_batch_pass<E, L, U, true, KT, TRON_LOSS_LR, S>, k_batch_pass<E, L, U, true, KT, TRON_LOSS_L2SVM, S>}};
    }
    return {{k_batch_pass<E, L, U, false, KT, TRON_LOSS_LR, S>, k_batch_pass<E, L, U, false, KT, TRON_LOSS_L2SVM, S>}};
    }
}

template <int KT, bool STREAM = false>
PassPair pass_for_shape(const Shape &s, bool vec)
{
    switch (s.L * 16 + s.E) {
    case 16 + 1: return pass_for<1, 1, KT, STREAM>(vec);
    case 16 + 2: return pass_for<2, 1, KT, STREAM>(vec);
    case 16 + 3: return pass_for<3, 1, KT, STREAM>(vec);
    case 16 + 4: return pass_for<4, 1, KT, STREAM>(vec);
    case 16 + 5: return pass_for<5, 1, KT, STREAM>(vec);
    case 16 + 6: return pass_for<6, 1, KT, STREAM>(vec);
    case 16 + 7: return pass_for<7, 1, KT, STREAM>(vec);
    case 16 + 8: return pass_for<8, 1, KT, STREAM>(vec);
    case 32 + 5: return pass_for<5, 2, KT, STREAM>(vec);
    case 32 + 6: return pass_for<6, 2, KT, STREAM>(vec);
    case 32 + 7: return pass_for<7, 2, KT, STREAM>(vec);
    case 32 + 8: return pass_for<8, 2, KT, STREAM>(vec);
    case 64 + 5: return pass_for<5, 4, KT, STREAM>(vec);
    case 64 + 6: return pass_for<6, 4, KT, STREAM>(vec);
    case 64 + 7: return pass_for<7, 4, KT, STREAM>(vec);
    case 64 + 8: return pass_for<8, 4, KT, STREAM>(vec);
    default: return {{nullptr, nullptr}};
    }
}

template <int DMAX, int KT, int RT, bool FG>
PassPair mfma_pass_pair(bool vec)
{
    if constexpr (KT == 8) {   // logistic problems only
        if (vec) return {{k_batch_pass_mfma<true, DMAX, KT, TRON_LOSS_LR, RT, FG>, nullptr}};
        return {{k_batch_pass_mfma<false, DMAX, KT, TRON_LOSS_LR, RT, FG>, nullptr}};
    } else {
        if (vec) return {{k_batch_pass_mfma<true, DMAX, KT, TRON_LOSS_LR, RT, FG>, k_batch_pass_mfma<true, DMAX, KT, TRON_LOSS_L2SVM, RT, FG>}};
        return {{k_batch_pass_mfma<false, DMAX, KT, TRON_LOSS_LR, RT, FG>, k_batch_pass_mfma<false, DMAX, KT, TRON_LOSS_L2SVM, RT, FG>}};
    }
}

template <int KT, int RT, bool FG>
PassPair mfma_pass_for(int64_t d)
{
    const bool vec = d % 2 == 0;
    if (d <= 16) return mfma_pass_pair<16, KT, RT, FG>(vec);
    if (d <= 24) return mfma_pass_pair<24, KT, RT, FG>(vec);
    return mfma_pass_pair<32, KT, RT, FG>(vec);
}

template <bool FG>
PassPair mfma_pass_select(int KT, int rt, int64_t d)
{
    if (rt == 64) return (KT == 8) ? mfma_pass_for<8, 64, FG>(d) : mfma_pass_for<16, 64, FG>(d);
    return (KT == 8) ? mfma_pass_for<8, 32, FG>(d) : mfma_pass_for<16, 32, FG>(d);
}

}  // namespace
}  // namespace tron

// ------------------------------------------------------------------ the handle
struct tron_batch {
    tron_dataset *ds = nullptr;
    int K = 0, KT = 0;
    int64_t ntiles = 0;
    uint64_t *member = nullptr;   // K planes of ntiles words
    uint64_t *Dbits = nullptr;    // K x 2 planes (L2-SVM active sets)
    double *Dval = nullptr;       // K x 2 x n (logistic D), allocated at the first logistic call
    tron::DriverState drv;
    double *partials = nullptr;           // K x (d+1) x grid
    tron::PassPair pass{{nullptr, nullptr}};
    size_t pass_lds[2] = {0, 0};          // dynamic LDS of the pass kernel per loss (the matrix-unit pass, tiles that come through LDS; 0 otherwise)
    // the matrix-unit pass for rounds in which no problem asks for function and gradient (null: none), with its own
    // dynamic LDS and number of resident workgroups per loss; grid_used = the workgroups of the pass launched last
    tron::PassPair pass_nofg{{nullptr, nullptr}};
    size_t pass_nofg_lds[2] = {0, 0};
    int grid_nofg[2] = {0, 0};
    int grid_pass[2] = {0, 0};            // workgroups of pass.fn per loss
    bool on_matrix_units[2] = {false, false};   // per loss: pass.fn is the matrix-unit kernel
    int grid_used = 0;
    int D_loss = -1;                      // loss whose D the buffers hold (-1: none)
};

namespace tron {
namespace {

// no_fg: the caller knows that no problem is in MODE_FG in this round
int launch_pass(tron_batch *b, int loss, bool no_fg = false)
{
    tron_dataset *ds = b->ds;
    ProfScope ps(ds, SLOT_BATCH_PASS);
    const int li = loss == TRON_LOSS_L2SVM ? 1 : 0;
    const bool lean = no_fg && b->pass_nofg.fn[li] != nullptr;
    const PassFn fn = lean ? b->pass_nofg.fn[li] : b->pass.fn[li];
    const size_t lds = lean ? b->pass_nofg_lds[li] : b->pass_lds[li];
    b->grid_used = lean ? b->grid_nofg[li] : b->grid_pass[li];
    int64_t n = ds->n, d = ds->d, ntiles = b->ntiles;
    const double *X = ds->X;
    const int8_t *y = ds->y8;
    const BatchCtl *ctl = b->drv.ctl;
    const uint64_t *member = b->member, *Din = b->Dbits;
    uint64_t *Dout = b->Dbits;
    double *Dval = b->Dval, *partials = b->partials;
    int K = b->K;
    void *args[] = {&n, &d, &X, &y, &ctl, &member, &Din, &Dout, &Dval, &ntiles, &partials, &K};
    TRON_HIP(hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(b->grid_used), dim3(kBlock), args, lds, ds->stream));
    return TRON_OK;
}

int launch_advance(tron_batch *b, const SolveParams &P, int64_t stamp)
{
    tron_dataset *ds = b->ds;
    ProfScope ps(ds, SLOT_BATCH_ADVANCE);
    hipLaunchKernelGGL(k_batch_advance, dim3(b->K), dim3(kAdvanceBlock), 0, ds->stream, ds->d, b->grid_used, b->partials, b->drv.ctl, b->drv.st, P,
                       P.trace_cap > 0 ? b->drv.trace_dev : nullptr, b->drv.host_dev, stamp);
    TRON_HIP(hipGetLastError());
    return TRON_OK;
}

int launch_begin(tron_dataset *ds, DriverState &drv, int K, int what, const double *IN, const double *C_host)
{
    BatchC Cs;
    for (int k = 0; k < kBatchMax; ++k) Cs.v[k] = (k < K) ? C_host[k] : 1.0;
    ProfScope ps(ds, SLOT_BATCH_ADVANCE);
    hipLaunchKernelGGL(k_batch_begin, dim3(K), dim3(kWave), 0, ds->stream, what, ds->d, IN, Cs, drv.ctl, drv.st);
    TRON_HIP(hipGetLastError());
    return TRON_OK;
}

// Enqueues rounds until every problem is idle: launch(stamp, no_fg), stamp = 1, 2, ...  The kernels write every problem's
// stamp and next mode into pinned memory, which the host polls while the device works: it keeps some rounds enqueued behind
// the last one it has seen (a round that finds every problem idle takes 2 us).  Copying the modes to the host and waiting for
// the stream every fourth round, as this replaces, took 40 us of a solve's 170 (20,000 x 24).
// It returns when every problem has its results, which come before the stamp that says so; the rounds behind the last one are then
// still to run (and find nothing to do).  So the numbers of the rounds go on from call to call: a stamp of an earlier call counts
// for nothing.
// ahead: the rounds kept enqueued.  Two where a round takes less than about 20 us (16 MB), for shorter ones the queue would
// run empty; one otherwise: 1M x 24 with six problems 321 us a solve with two, the last of which keep the stream busy for 18.
// exact: wait for every round before the next, and tell the launch when no problem asks for function and gradient.
template <class Launch>
int drive_rounds(tron_dataset *ds, DriverState &drv, int K, int64_t round_cap, bool exact, Launch launch)
{
    const int64_t before = drv.rounds, ahead = exact ? 0 : (double)ds->n * (double)ds->d * 8.0 > 16e6 ? 1 : 2;
    int64_t launched = 0;
    for (unsigned spins = 0;;) {
        int64_t seen = INT64_MAX;
        bool live = false, fg = false;
        for (int k = 0; k < K; ++k) {
            const int64_t v = __atomic_load_n(&drv.host->stamp[k], __ATOMIC_ACQUIRE), round = std::max<int64_t>((v >> 2) - before, 0);
            seen = std::min(seen, round);
            live |= round == 0 || (v & 3) != MODE_IDLE;
            fg |= (v & 3) == MODE_FG;
        }
        if (!live) return TRON_OK;
        if (launched < seen + ahead + 1) {
            if (launched > round_cap + ahead) { set_error("internal: problems still running after the round limit"); return TRON_ESTATE; }
            ++launched;
            drv.rounds += 1;
            TRON_TRY(launch(drv.rounds, exact && launched > 1 && !fg));
            spins = 0;
            continue;
        }
        if ((++spins & 1023u) != 0) { __builtin_ia32_pause(); continue; }
        // nothing new for a while: make sure that the kernels are still running
        const hipError_t e = hipStreamQuery(ds->stream);
        (void)hipGetLastError();
        if (e != hipSuccess && e != hipErrorNotReady) return hip_fail(e, "hipStreamQuery", __FILE__, __LINE__);
        if (e == hipSuccess) {
            int64_t last = INT64_MAX;
            for (int k = 0; k < K; ++k) last = std::min(last, __atomic_load_n(&drv.host->stamp[k], __ATOMIC_ACQUIRE) >> 2);
            if (last < drv.rounds) { set_error("internal: a round has ended without its stamp"); return TRON_ESTATE; }
        }
        std::this_thread::yield();
    }
}

// what problem k's results say
void fill_result(const DriverState &drv, int k, int cap, tron_result &r)
{
    const ProbScalars &sc = drv.host->sc[k];
    r.f = sc.f; r.gnorm = sc.gnorm; r.gnorm0 = sc.gnorm0;
    r.outer_iters = sc.outer; r.cg_iters_total = sc.cg_total; r.n_fun = sc.n_fun; r.n_grad = sc.n_grad; r.n_hv = sc.n_hv;
    r.converged = sc.converged;
    r.trace_len = sc.trace_len < r.trace_cap ? sc.trace_len : r.trace_cap;
    if (r.trace_len > 0) memcpy(r.trace, drv.trace + (size_t)k * cap, sizeof(tron_trace_rec) * r.trace_len);
}

// A problem needs at most 3 + max_outer (max_cg + 2) rounds (one more per iterate with a preconditioner).
int64_t round_limit(const tron_params &Q) { return 3 + (int64_t)Q.max_outer * ((int64_t)Q.max_cg + 2); }

int ensure_D(tron_batch *b, int loss)
{
    if (loss == TRON_LOSS_LR && !b->Dval) {
        // zero once: a pass only ever writes D of a problem's own rows, the others stay zero
        const size_t bytes = sizeof(double) * 2 * (size_t)b->K * (size_t)b->ds->n;
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&b->Dval), bytes));
        TRON_HIP(hipMemsetAsync(b->Dval, 0, bytes, b->ds->stream));
    }
    return TRON_OK;
}

bool bad_C(const tron_batch *b, const double *C_host)
{
    for (int k = 0; k < b->K; ++k)
        if (!(C_host[k] > 0.0) || !std::isfinite(C_host[k])) return true;
    return false;
}

// one single product for every problem: begin, pass, advance, results to OUT (K*d) and scal_host (K)
int one_shot(tron_batch *b, int what, int loss, const double *C_host, const double *IN, double *OUT, double *scal_host)
{
    tron_dataset *ds = b->ds;
    SolveParams P{};
    P.loss = loss;
    P.out = OUT;
    TRON_TRY(launch_begin(ds, b->drv, b->K, what, IN, C_host));
    TRON_TRY(launch_pass(b, loss, what == BEGIN_HV));
    TRON_TRY(launch_advance(b, P, ++b->drv.rounds));
    // a problem's stamp comes after its results
    auto arrived = [&]() {
        for (int k = 0; k < b->K; ++k)
            if (__atomic_load_n(&b->drv.host->stamp[k], __ATOMIC_ACQUIRE) >> 2 != b->drv.rounds) return false;
        return true;
    };
    for (unsigned spins = 1; !arrived(); ++spins) {
        if ((spins & kSpinsPerQuery) == 0 && hipStreamQuery(ds->stream) != hipErrorNotReady) {
            (void)hipGetLastError();
            TRON_HIP(hipStreamSynchronize(ds->stream));
            break;
        }
        __builtin_ia32_pause();
    }
    if (scal_host)
        for (int k = 0; k < b->K; ++k) scal_host[k] = b->drv.host->sc[k].out_scal;
    return TRON_OK;
}

}  // namespace
}  // namespace tron

using namespace tron;

extern "C" void tron_batch_destroy(tron_batch *b)
{
    if (!b) return;
    if (b->ds) hipStreamSynchronize(b->ds->stream);
    hipFree(b->member); hipFree(b->Dbits); hipFree(b->Dval); hipFree(b->partials);
    b->drv.release();
    delete b;
}

static int batch_create_impl(tron_dataset *ds, int K, const uint32_t *member, int mem, tron_batch **out)
{
    *out = nullptr;
    if (!ds->dense || ds->d > kVecPad) {
        set_error("tron_batch_create: needs a dense dataset with d <= %d", kVecPad);
        return TRON_EINVAL;
    }
    const int64_t n = ds->n, d = ds->d;
    if (mem == TRON_MEM_HOST)
        for (int64_t i = 0; i < n; ++i)
            if ((member[i] >> K) != 0u) { set_error("tron_batch_create: member[%lld] has a bit at or above K", (long long)i); return TRON_EINVAL; }
    Shape s;
    if (!pick_shape(d, s) || s.L > 4) { set_error("tron_batch_create: internal: no tile shape for d = %lld", (long long)d); return TRON_EINVAL; }
    tron_batch *b = new (std::nothrow) tron_batch();
    if (!b) { set_error("out of host memory"); return TRON_ENOMEM; }
    b->ds = ds;
    b->K = K;
    b->KT = (K <= 4) ? 4 : 8;
    b->ntiles = (n + kWave - 1) / kWave;
    const bool vec = (s.E % 2 == 0) && (d % 2 == 0);
    // up to 8 problems: the pass on the vector units (4 or 8 problem slots), unless the matrix units take it (below)
    b->pass = (b->KT == 4) ? pass_for_shape<4>(s, vec) : pass_for_shape<8>(s, vec);
    auto fail = [&](int rc) { tron_batch_destroy(b); return rc; };
#define TRON_B(expr) do { hipError_t e__ = (expr); if (e__ != hipSuccess) return fail(hip_fail(e__, #expr, __FILE__, __LINE__)); } while (0)
    if (!b->pass.fn[0]) { set_error("tron_batch_create: internal: no kernel for E=%d L=%d", s.E, s.L); return fail(TRON_EINVAL); }
    // The pass as matrix instructions (8 or 16 problem columns; the tile of X of every wavefront in LDS, and where logistic
    // function / gradient requests are served the exchange area), chosen per loss: above eight problems always, and for logistic problems
    // from seven on where a lane has eight columns, whose accumulators do not fit the registers of the vector kernel, from eight on over matrices
    // above 288 MB, where neither is the faster one throughout.  us a function-gradient / Hessian call of 5, 6, 7, 8 problems over 10M rows, vector
    // units against matrix units.  L2-SVM, 24 columns: 395 418 452 485 / 325 333 346 364 against 531 529 531 535 / 400 404 406 413; 12 columns, 8 problems:
    // 320 / 200 against 383 / 261; where the tiles have no room in LDS, 8 problems, and a solve with them: 1M x 32 103 / 84, 411 against 99 / 93, 431; 4M x 29
    // 288 / 217, 1237 against 276 / 231, 1270; 4M x 32, the worst for the vector units, 283 / 218, 1222 against 258 / 217, 1183.  Logistic, 24 columns: 643 687 737 785 / 436 441 463 483 against 684 701 739 763 / 490 492 498 507; 30 columns: 726 766
    // 823 991 / 560 564 722 910 against 764 782 820 845 / 562 575 580 584; 8 problems, 12 columns: 563 / 300 against 553 / 338; 4M x 16: 280 / 160 against
    // 261 / 170; 1M x 24: 93 / 70 against 106 / 75.
    const int mfma_from[2] = {s.L == 4 && s.E == 8 ? 7 : read_once(n, d) ? 8 : 9, 9};   // logistic, L2-SVM
    const int dmax = d <= 16 ? 16 : (d <= 24 ? 24 : 32);
    const size_t floor_lds = sizeof(double) * kWavesPerBlock * 32 * 16;   // the final sums of the four wavefronts
    for (int l = 0; l < 2; ++l) {
        b->on_matrix_units[l] = K > 8 || g_tuning.batch_mfma > 0 || (g_tuning.batch_mfma < 0 && K >= mfma_from[l]);
        if (!b->on_matrix_units[l]) continue;
        const int KTm = l == 0 && K <= 8 ? 8 : 16;
        // half tiles (measured: as fast or faster than whole tiles for both losses, 3 to 12% at 12 problems)
        const int rt = g_tuning.batch_mfma_rows != 0 ? (int)g_tuning.batch_mfma_rows : 32;
        b->pass.fn[l] = mfma_pass_select<true>(KTm, rt, d).fn[l];
        b->pass_lds[l] = sizeof(double) * kWavesPerBlock * (size_t)mfma_wave_doubles(dmax, l == 0 ? K : 0, rt);
        if (b->pass_lds[l] < floor_lds) b->pass_lds[l] = floor_lds;
        TRON_B(hipFuncSetAttribute(reinterpret_cast<const void *>(b->pass.fn[l]), hipFuncAttributeMaxDynamicSharedMemorySize, (int)b->pass_lds[l]));
        if (g_tuning.batch_lean != 0) {
            // rounds without function / gradient requests: three to five wavefronts per SIMD; half tiles here too (with whole ones the L2-SVM
            // kernel does not fit its registers from 17 columns on: 12 problems over 4M x 17 530 us a call, 189 with half tiles)
            const int rt_lean = g_tuning.batch_mfma_rows != 0 ? (int)g_tuning.batch_mfma_rows : 32;
            b->pass_nofg.fn[l] = mfma_pass_select<false>(KTm, rt_lean, d).fn[l];
            b->pass_nofg_lds[l] = sizeof(double) * kWavesPerBlock * (size_t)mfma_wave_doubles(dmax, 0, rt_lean);
            if (b->pass_nofg_lds[l] < floor_lds) b->pass_nofg_lds[l] = floor_lds;
            TRON_B(hipFuncSetAttribute(reinterpret_cast<const void *>(b->pass_nofg.fn[l]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)b->pass_nofg_lds[l]));
        }
    }
    // resident workgroups of a pass: all of them hold their accumulators for the whole pass
    int cus = 0;
    TRON_B(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ds->device));
    const int64_t by_tiles = (b->ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
    auto resident = [&](PassFn fn, size_t lds, int *out) -> int {
        int pc = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&pc, reinterpret_cast<const void *>(fn), kBlock, lds);
        if (e != hipSuccess) return hip_fail(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor", __FILE__, __LINE__);
        int64_t gl = (int64_t)cus * (pc < 1 ? 1 : pc);
        if (g_tuning.batch_grid > 0) gl = g_tuning.batch_grid;
        if (gl > by_tiles) gl = by_tiles;
        if (gl < 1) gl = 1;
        *out = (int)gl;
        return TRON_OK;
    };
    int64_t grid_max = 1;
    for (int l = 0; l < 2; ++l) {
        int rc = resident(b->pass.fn[l], b->pass_lds[l], &b->grid_pass[l]);
        if (rc == TRON_OK && b->pass_nofg.fn[l]) rc = resident(b->pass_nofg.fn[l], b->pass_nofg_lds[l], &b->grid_nofg[l]);
        if (rc != TRON_OK) return fail(rc);
        if (b->grid_pass[l] > grid_max) grid_max = b->grid_pass[l];
        if (b->grid_nofg[l] > grid_max) grid_max = b->grid_nofg[l];
    }
    if (!b->on_matrix_units[0] && !b->on_matrix_units[1]) {
        // the two vector kernels share one grid (the larger residency), as they always have
        b->grid_pass[0] = b->grid_pass[1] = (int)grid_max;
    }
    if (tiles_stream(s.L) && read_once(n, d)) {
        const PassPair streamed = b->KT == 4 ? pass_for_shape<4, true>(s, vec) : pass_for_shape<8, true>(s, vec);
        const size_t through = TileStream<1, 2, 2, false>::bytes(d, kWavesPerBlock);
        for (int l = 0; l < 2; ++l) {
            if (b->on_matrix_units[l] || !streamed.fn[l]) continue;
            TRON_B(hipFuncSetAttribute(reinterpret_cast<const void *>(streamed.fn[l]), hipFuncAttributeMaxDynamicSharedMemorySize, (int)through));
            int at_once = 0;
            TRON_B(hipOccupancyMaxActiveBlocksPerMultiprocessor(&at_once, reinterpret_cast<const void *>(streamed.fn[l]), kBlock, through));
            if (at_once < 2) continue;   // from 29 (more than four problems) or 31 columns (logistic) on the tiles leave room for one workgroup
            b->pass.fn[l] = streamed.fn[l];
            b->pass_lds[l] = through;
            const int rc = resident(streamed.fn[l], through, &b->grid_pass[l]);
            if (rc != TRON_OK) return fail(rc);
            if (b->grid_pass[l] > grid_max) grid_max = b->grid_pass[l];
        }
    }
    b->grid_used = b->grid_pass[1];
    TRON_B(hipMalloc(reinterpret_cast<void **>(&b->member), sizeof(uint64_t) * (size_t)K * (size_t)b->ntiles));
    TRON_B(hipMalloc(reinterpret_cast<void **>(&b->Dbits), sizeof(uint64_t) * 2 * (size_t)K * (size_t)b->ntiles));
    {
        const int rc = b->drv.create(K, ds->stream);
        if (rc != TRON_OK) return fail(rc);
    }
    TRON_B(hipMalloc(reinterpret_cast<void **>(&b->partials), sizeof(double) * (size_t)K * (size_t)(d + 1) * (size_t)grid_max));
    TRON_B(hipMemsetAsync(b->Dbits, 0, sizeof(uint64_t) * 2 * (size_t)K * (size_t)b->ntiles, ds->stream));
    // membership words; a device-side check of the unused bits for device input
    uint32_t *staged = nullptr;
    int *bad = nullptr;
    TRON_B(hipMalloc(reinterpret_cast<void **>(&bad), sizeof(int)));
    hipError_t e = hipMemsetAsync(bad, 0, sizeof(int), ds->stream);
    const uint32_t *src = member;
    if (e == hipSuccess && mem == TRON_MEM_HOST) {
        e = hipMalloc(reinterpret_cast<void **>(&staged), sizeof(uint32_t) * (size_t)n);
        if (e == hipSuccess) e = hipMemcpyAsync(staged, member, sizeof(uint32_t) * (size_t)n, hipMemcpyHostToDevice, ds->stream);
        src = staged;
    }
    int bad_host = 0;
    if (e == hipSuccess) {
        int64_t g = (b->ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
        if (g > kMaxGrid) g = kMaxGrid;
        hipLaunchKernelGGL(k_member_planes, dim3((int)g), dim3(kBlock), 0, ds->stream, n, K, src, b->ntiles, b->member, bad);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&bad_host, bad, sizeof(int), hipMemcpyDeviceToHost, ds->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ds->stream);
    hipFree(staged);
    hipFree(bad);
    if (e != hipSuccess) return fail(hip_fail(e, "membership words", __FILE__, __LINE__));
    if (bad_host) { set_error("tron_batch_create: a member word has a bit at or above K"); return fail(TRON_EINVAL); }
#undef TRON_B
    *out = b;
    return TRON_OK;
}

extern "C" int tron_batch_create(tron_dataset *ds, int K, const uint32_t *member, int mem, tron_batch **out)
{
    if (out) *out = nullptr;
    if (!ds || !out || !member || K < 1 || K > kBatchMax || (mem != TRON_MEM_HOST && mem != TRON_MEM_DEVICE)) {
        set_error("tron_batch_create: bad argument (need a handle, 1 <= K <= %d, member, mem in {0,1}, out)", kBatchMax);
        return TRON_EINVAL;
    }
    return batch_create_impl(ds, K, member, mem, out);
}

extern "C" int tron_batch_fun_grad(tron_batch *b, int loss, const double *C_host, const double *W_dev, double *f_host,
                                   double *G_dev)
{
    if (!b || !C_host || !W_dev || !f_host || (loss != TRON_LOSS_LR && loss != TRON_LOSS_L2SVM) || bad_C(b, C_host)) {
        set_error("tron_batch_fun_grad: bad argument (null batch/C/W/f, unknown loss, or some C <= 0)");
        return TRON_EINVAL;
    }
    TRON_TRY(ensure_D(b, loss));
    TRON_TRY(one_shot(b, BEGIN_FG, loss, C_host, W_dev, G_dev, f_host));
    b->D_loss = loss;
    return TRON_OK;
}

extern "C" int tron_batch_hv(tron_batch *b, const double *C_host, const double *V_dev, double *HV_dev, double *vHv_host)
{
    if (!b || !C_host || !V_dev || !HV_dev || V_dev == HV_dev || bad_C(b, C_host)) {
        set_error("tron_batch_hv: bad argument (null batch/C/V/HV, V aliases HV, or some C <= 0)");
        return TRON_EINVAL;
    }
    if (b->D_loss < 0) { set_error("tron_batch_hv: no cached D; call tron_batch_fun_grad first"); return TRON_ESTATE; }
    return one_shot(b, BEGIN_HV, b->D_loss, C_host, V_dev, HV_dev, vHv_host);
}

extern "C" int tron_batch_solve(tron_batch *b, const tron_params *params, const double *C_host, double *W_dev,
                                tron_result *res, int *status_host)
{
    if (!b || !params || !C_host || !W_dev || !res) { set_error("tron_batch_solve: null argument"); return TRON_EINVAL; }
    const tron_params &Q = *params;
    if ((Q.loss != TRON_LOSS_LR && Q.loss != TRON_LOSS_L2SVM) || bad_C(b, C_host) || !(Q.eps > 0.0) || Q.max_outer < 1 ||
        Q.max_cg < 1 || !(Q.cg_xi > 0.0) || !(Q.cg_xi < 1.0) || !(Q.precond_blend >= 0.0) || !(Q.precond_blend <= 1.0)) {
        set_error("tron_batch_solve: bad parameter (loss, every C > 0, eps > 0, max_outer >= 1, max_cg >= 1, 0 < cg_xi < 1, "
                  "0 <= precond_blend <= 1)");
        return TRON_EINVAL;
    }
    int cap = 0;
    for (int k = 0; k < b->K; ++k) {
        if (res[k].trace_cap < 0 || (res[k].trace_cap > 0 && !res[k].trace)) { set_error("tron_batch_solve: bad trace of problem %d", k); return TRON_EINVAL; }
        if (res[k].trace_cap > cap) cap = res[k].trace_cap;
    }
    tron_dataset *ds = b->ds;
    TRON_TRY(ensure_D(b, Q.loss));
    if (cap > Q.max_outer) cap = Q.max_outer;   // one record per outer iteration
    TRON_TRY(b->drv.ensure_trace(b->K, cap));
    const SolveParams P{Q.loss, Q.max_outer, Q.max_cg, cap, Q.eps, Q.cg_xi, W_dev, Q.precond_blend};
    b->D_loss = -1;
    TRON_TRY(launch_begin(ds, b->drv, b->K, BEGIN_SOLVE, W_dev, C_host));
    // Rounds of large matrices that have the lean matrix-unit kernel: worth knowing before each whether it will do.
    const int li = Q.loss == TRON_LOSS_L2SVM ? 1 : 0;
    const bool exact = b->pass_nofg.fn[li] != nullptr && (double)ds->n * (double)ds->d * 8.0 >= 4e8;
    TRON_TRY(drive_rounds(ds, b->drv, b->K, round_limit(Q), exact, [&](int64_t stamp, bool no_fg) -> int {
        TRON_TRY(launch_pass(b, Q.loss, no_fg));
        return launch_advance(b, P, stamp);
    }));
    int overall = TRON_OK;
    for (int k = 0; k < b->K; ++k) {
        fill_result(b->drv, k, cap, res[k]);
        const int status = b->drv.host->sc[k].status;
        if (status_host) status_host[k] = status;
        if (status != TRON_OK) overall = TRON_EMAXITER;
    }
    b->D_loss = Q.loss;
    return overall;
}

// ------------------------------------------------------------------ one problem, driven from the device
// tron_solve for a dense matrix with d <= 32 in one launch (k_dense_solve), or where its workgroups cannot all be resident in a
// launch per round, so that no scalar is waited for by the host inside an iteration and no vector kernels run between the passes.
namespace tron {

int DriverState::create(int K, hipStream_t stream)
{
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&ctl), sizeof(BatchCtl)));
    TRON_HIP(hipMalloc(reinterpret_cast<void **>(&st), sizeof(ProbState) * K));
    TRON_HIP(hipHostMalloc(reinterpret_cast<void **>(&host), sizeof(BatchHost), hipHostMallocMapped));
    TRON_HIP(hipHostGetDevicePointer(reinterpret_cast<void **>(&host_dev), host, 0));
    memset(host, 0, sizeof(BatchHost));
    TRON_HIP(hipMemsetAsync(ctl, 0, sizeof(BatchCtl), stream));
    TRON_HIP(hipMemsetAsync(st, 0, sizeof(ProbState) * K, stream));
    return TRON_OK;
}

int DriverState::ensure_trace(int K, int cap)
{
    if (cap <= trace_cap) return TRON_OK;
    if (trace) hipHostFree(trace);
    trace = nullptr;
    trace_cap = 0;
    TRON_HIP(hipHostMalloc(reinterpret_cast<void **>(&trace), sizeof(tron_trace_rec) * (size_t)K * (size_t)cap, hipHostMallocMapped));
    TRON_HIP(hipHostGetDevicePointer(reinterpret_cast<void **>(&trace_dev), trace, 0));
    trace_cap = cap;
    return TRON_OK;
}

void DriverState::release()
{
    hipFree(ctl);
    hipFree(st);
    if (host) hipHostFree(host);
    if (trace) hipHostFree(trace);
    *this = DriverState();
}

int dense_device_solve(tron_dataset *ds, const tron_params &Q, double *w_dev, tron_result *res)
{
    if (!ds->driver) {
        ds->driver = new (std::nothrow) DriverState();
        if (!ds->driver) { set_error("out of host memory"); return TRON_ENOMEM; }
    }
    DriverState &drv = *ds->driver;
    if (!drv.host) {
        const int rc = drv.create(1, ds->stream);
        if (rc != TRON_OK) { drv.release(); return rc; }
    }
    const int cap = std::min(res->trace_cap, Q.max_outer);
    TRON_TRY(drv.ensure_trace(1, cap));
    const SolveParams P{Q.loss, Q.max_outer, Q.max_cg, cap, Q.eps, Q.cg_xi, w_dev, Q.precond_blend};
    ds->have_D = false;
    ds->hat_slot = -1;   // both D buffers are overwritten
    const double C = Q.C;
    bool done = false;
    const int grid = dense_round_grid(ds->n, ds->d, Q.loss);
    std::optional<ResidentShare> share;
    if (resident_possible(ds, grid)) share.emplace(ds, grid, ds->resident.try_it(g_tuning.solve_wait_us) ? 1 : 0);
    if (share && share->granted()) {
        drv.host->finished = 0;
        TRON_TRY(dense_solve_launch(ds, P, drv, 0, w_dev, C));
        // With the stamp everything is there that the call returns; the stream's own wait would take some microseconds more.
        auto ended = [&]() { return __atomic_load_n(&drv.host->finished, __ATOMIC_ACQUIRE) != 0; };
        for (unsigned spins = 1; !ended(); ++spins) {
            if ((spins & kSpinsPerQuery) == 0 && hipStreamQuery(ds->stream) != hipErrorNotReady) break;
            __builtin_ia32_pause();
        }
        if (!ended()) {
            (void)hipGetLastError();
            TRON_HIP(hipStreamSynchronize(ds->stream));
        }
        done = ended();   // otherwise workgroups gave up waiting for others before the first of them had the result; w0 is as it was
        ds->resident.ended(done);
        share->give_back();
    }
    if (!done) {
        TRON_TRY(launch_begin(ds, drv, 1, BEGIN_SOLVE, w_dev, &C));
        TRON_TRY(drive_rounds(ds, drv, 1, round_limit(Q), false, [&](int64_t stamp, bool) -> int { return dense_solve_launch(ds, P, drv, stamp, nullptr, C); }));
    }
    fill_result(drv, 0, cap, *res);
    // D at the final iterate, in the layout of the single-problem calls (one bit per row in 64-bit words for the L2-SVM, fp64 per
    // row for the logistic loss)
    ds->Dcur = drv.host->sc[0].dcur;
    ds->have_D = true;
    for (int slot = 0; slot < 2; ++slot) {
        ds->D_is_mask[slot] = (Q.loss == TRON_LOSS_L2SVM);
        ds->active_frac[slot] = 1.0;   // not counted here: the Hessian pass then reads every row, which is always right
    }
    return drv.host->sc[0].status;
}

void dense_device_release(tron_dataset *ds)
{
    if (ds->driver) ds->driver->release();
    delete ds->driver;
    ds->driver = nullptr;
}

}  // namespace tron
