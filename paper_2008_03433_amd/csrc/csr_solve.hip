// A whole sparse solve (Algorithm 1 of the paper with Steihaug's truncated CG) in one launch whose workgroups wait for each other.
//
// A solve of a small matrix is a chain of dependent steps, each of a few microseconds: as launches, three or four per CG iteration
// and four per evaluation, it spends most of its time between them and on fetching the matrix again for every product.  Here a
// step is one product with X or with X^T, and between two steps lies one barrier over the grid (grid_sync.h):
//   with X:   margins of a trial point -> loss terms; or u = D (X p), and p.Hp = p.p + C sum u (X p)
//   with X^T: the gradient; or Hp, and in the same pass the step s, the residual r and the trial point
// A CG iteration is two steps: the direction p = z + beta p (z = r / M) is formed where it is gathered, from pairs (z, p) of the
// iteration before, so that nothing waits for beta alone.
//
// What other workgroups read is written with store_shared and read with ordinary loads, which L1 and L2 may keep: no load may find a line that
// was filled before the last writing.  Pairs and u go to kRing places in turn: each time the places have been used up, one wavefront
// of every workgroup invalidates what its caches hold (an acquire of device scope; a barrier of the workgroup behind it covers the other
// wavefronts), and between two such fences a place is written once and read after that.  The trial point and D (for the
// preconditioner) lie in the same places every time, with a fence of their own before the product that gathers from them.  A line that a
// workgroup writes a part of must not come back with old neighbours: see store_shared.  Everything else that changes belongs to one workgroup, the one
// whose chunk holds the row's first entry (for rows longer than a chunk: workgroup l mod the grid for the l-th), and is its own to read.
//
// Latencies bound it: a step is some 6 us with 49 chunks, 13 with 513 -- entries and the first gathers from beyond L2 2 to 5 us, row
// sums and stores 1.5, long rows 2, the barrier 1.5 to 2.5, sums over the grid and the next decision 1.5.  Two chunks of 256 threads a
// workgroup leave 256 registers a thread, which the fetched chunk, the row's vectors and nine sums fill; three chunks (168 registers)
// are no faster although 513 chunks then need no second round, four spill.  us a solve, driven by the host / here: 100,000 entries
// 227 / 117, 264,000 230 / 139, 480,000 245 / 172, 1.05M with Zipf-distributed columns 955 / 864 (more at kMaxRounds).  The error of w
// against sums in extended precision, over 576 solves of six shapes, is 0.95 +- 0.05 of the host-driven solve's (geometric mean of the ratios),
// although p.p, p.Mp and s.Mp come from recurrences.
// (Solves of several threads that together need more than the GPU: see ResidentShare in common.h, and PART_CHUNKS below.)
#include <cmath>
#include <new>
#include <thread>

#include "csr_chunk.h"
#include "grid_sync.h"

namespace tron {

constexpr int kTeam = kBlock;        // threads that share a chunk
constexpr int kMaxTeams = 2;         // chunks a workgroup has in hand
constexpr int kRing = 4;   // (8: no faster; the invalidation costs 1.4 us)
constexpr int kSums = 9;
constexpr int kPlainRows = 2048;     // most rows of a chunk: plain layout (a place each in LDS), segments
constexpr int kSegRows = 4096;
constexpr int kTeamLds = kProdDoubles + kPlainRows;   // (segments: 9/8 kChunk products, later the sums)
static_assert(kOutOffset + kChunk / 8 * 9 <= kTeamLds, "products of a chunk of segments");
constexpr int kMaxResidentGrid = 256;
constexpr int kLine = 16;            // words of 8 bytes
// Results of up to so many columns are copied out by the first workgroup, longer ones by a copy operation behind the launch.  us a solve of 1M
// entries, workgroup / operation: 5,000 columns 457 / 464, 12,000 469 / 470, 24,000 492 / 488, 47,000 523 / 503, 100,000 612 / 557.
constexpr int64_t kOutInKernel = 12'288;
constexpr int kStepsPerLaunch = 512;         // some milliseconds; a longer solve goes on in another launch

// one orientation of the matrix (see CsrPlan)
struct ChunkPlan {
    const int32_t *col;
    const double *val;
    const int32_t *row_lo;
    const int64_t *rowptr;      // plain
    const int4 *chunk_tab;      // segments
    const uint8_t *flags;
    const int32_t *row_seg;
    const int2 *chunk_long;
    const int4 *long_row;
    uint64_t *pieces;           // of the rows longer than a chunk, one per chunk and then one per such row; kEmpty until it is there
    int64_t stored;
    int nchunks, nlong;
};

constexpr uint64_t kEmpty = 0x7ff4dead00c0ffeeull;   // a NaN that no arithmetic returns

enum { STEP_END = 0, STEP_START, STEP_ZERO, STEP_TRIAL, STEP_CG,   // products with X
       STEP_START_G, STEP_ZERO_G, STEP_TRIAL_G, STEP_HV, STEP_DIAG, STEP_RESTART };   // with X^T, or (the last) none
__device__ __forceinline__ bool with_x(int step) { return step <= STEP_CG; }

struct RowTerms { double alpha, zhat, D; };

// A call, so that the coefficients of the logistic terms are not kept in registers through all steps
template <int LOSS>
__device__ __noinline__ RowTerms row_terms(double z, double y)
{
    RowTerms t;
    loss_terms_dev<LOSS>(z, y, t.alpha, t.zhat, t.D);
    return t;
}

// The state of the solve: every workgroup's own, all the same.
struct CsrState {
    int step, first_diag, it, onb, cur, dcur, outer, cg_total, n_fun, n_grad, n_hv, status, converged, trace_len;
    int turn;                // whose lines the step uses
    int na, nb;              // places used so far by the results of products with X, by those with X^T
    int pair_at;             // where the pairs lie
    double f, fnew, gnorm, gnorm0, gscaled, delta, rr, tol, beta, length, ww, pred, snorm, pp, pMp, sMp, ss;   // length: of the step along p
};

// What the host reads (pinned memory, kept with the scalars)
constexpr int kHostRecords = 32;
// The others go to device memory, as many places as the caller has, which stay with the handle: 64 MB at most.  Solves for more records are driven by
// the host, which writes them to the caller's array itself.
constexpr int kMaxRecords = 1 << 20;
struct CsrHost {
    CsrState st;
    tron_trace_rec trace[kHostRecords];
    int64_t stamp;   // launches that have ended with all workgroups together
    int64_t step;    // a launch per step: the last one that has begun
};

// The rest of what the kernel is told.  It copies this to LDS: kept in registers through all steps it would leave too few of them.
struct CsrSolveArgs {
    int64_t n, d;
    const double *y;
    double *D[2];
    double *pairs[kRing], *u[kRing], *point;
    double *w[2], *g[2], *s, *r, *M;
    double *sums;            // 2 x kSums x kMaxResidentGrid, for even and odd steps
    uint64_t *lines;         // three turns of kSyncFlat lines, one of a workgroup's sums each
    const double *w0;
    double *out;             // null: the host copies
    int loss, max_outer, max_cg, trace_cap, resume, steps, turn;
    double C, eps, xi, blend;
    GridSync sync;
    CsrState *state;
    CsrHost *host;
    tron_trace_rec *trace;
    int64_t stamp;
    double *lanes, *waves;   // a launch per step: what PART_CHUNKS leaves for PART_LONG, see there
};

// A chunk as a thread holds it before it multiplies: its eight entries, and of the first row it will finish what is needed
struct Chunk {
    int c[8];
    v2d v[4];
    unsigned flags;
    int lo, hi, seg, k0, k1;
    int4 tab;
    int2 lr;
};

// lanes that share a row's sum in the plain layout
__device__ __forceinline__ int lanes_per_row(int nrows)
{
    // the largest power of two up to 64 of which nrows fit into a team
    const int most = kTeam / (nrows > 1 ? nrows : 1);
    return most >= kWave ? kWave : most > 1 ? 1 << (31 - __clz(most)) : 1;
}

template <bool SEG>
__device__ __forceinline__ void load_chunk(const ChunkPlan &P, int chunk, int tid, Chunk &h)
{
    h.lo = h.hi = 0;
    h.flags = 0u;
    h.seg = -1;
    h.k0 = h.k1 = 0;
    h.tab = make_int4(0, 0, 0, 0);
    h.lr = make_int2(-1, -1);
#pragma unroll
    for (int e = 0; e < 8; ++e) h.c[e] = 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) h.v[m] = v2d{0.0, 0.0};
    if (chunk >= P.nchunks) return;
    const int64_t start = (int64_t)chunk * kChunk;
    if constexpr (SEG) {
        // Entries tid, tid + 256, ...: neighbouring lanes have neighbouring entries, which in the long rows gather from the same lines.
        // (See col_pos and val_pos in kernels_csr.hip for where they are.)
        const int32_t *col = P.col + start + (tid >> 2 & 1) * (kChunk / 2) + (tid >> 3) * 4 + (tid & 3);
        const double *val = P.val + start + (tid >> 1 & 3) * kQuarter + (tid >> 3) * 2 + (tid & 1);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            h.c[e] = col[e * (kTeam / 2)];
            h.v[e / 2][e % 2] = val[e * (kTeam / 4)];
        }
        h.flags = P.flags[(int64_t)chunk * kTeam + tid];
        h.lo = P.row_lo[chunk];
        h.hi = P.row_lo[chunk + 1];
        h.tab = P.chunk_tab[chunk];
        h.lr = P.chunk_long[chunk];
        if (h.lo + tid < h.hi) h.seg = P.row_seg[h.lo + tid];
    } else {
        h.lo = P.row_lo[chunk];
        h.hi = P.row_lo[chunk + 1];
        if (start + kChunk <= P.stored) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int64_t k = start + m * kQuarter + tid * 2;
                const v2i q = *reinterpret_cast<const v2i *>(P.col + k);
                h.c[2 * m] = q.x;
                h.c[2 * m + 1] = q.y;
                h.v[m] = *reinterpret_cast<const v2d *>(P.val + k);
            }
        } else {
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int64_t k = start + m * kQuarter + tid * 2 + e;
                    if (k < P.stored) {
                        h.c[2 * m + e] = P.col[k];
                        h.v[m][e] = P.val[k];
                    }
                }
        }
        const int row = h.lo + tid / lanes_per_row(h.hi - h.lo);
        if (row < h.hi) {
            h.k0 = (int)(P.rowptr[row] - start);
            h.k1 = (int)(P.rowptr[row + 1] - start);
        }
    }
}

enum { GATHER_NONE = 0, GATHER_ONE, GATHER_PAIR };

// out[...] = the sums of the chunk's rows (SEG: of its segments, by number; plain: by row), behind a barrier.  SEG: piece = the sum
// of a row's piece that began in an earlier chunk.
template <bool SEG>
__device__ __forceinline__ void chunk_sums(const ChunkPlan &P, int chunk, int tid, const Chunk &h, int how, const double *x, double beta, bool square,
                                           double *lds, double *piece)
{
    double q[8];
    if (how == GATHER_PAIR) {
        v2d t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = reinterpret_cast<const v2d *>(x)[(uint32_t)h.c[e]];
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = fma(beta, t[e].y, t[e].x);
    } else if (how == GATHER_ONE) {
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = x[(uint32_t)h.c[e]];
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = 0.0;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const double v = h.v[e / 2][e % 2];
        q[e] *= square ? v * v : v;
    }
    if constexpr (SEG) {
        double cin;
        int idx0;
        double *prod = lds + kOutOffset;   // one place more after every eight, so that eight in a row are read without bank conflicts
#pragma unroll
        for (int e = 0; e < 8; ++e) prod[e * (kTeam + kTeam / 8) + tid + tid / 8] = q[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = prod[9 * tid + e];
        runs_from_regs(lds, tid, h.flags, q, cin, idx0);
        double *out = lds + kOutOffset;
        int i = idx0 - (h.tab.z > 0 ? 1 : 0);
        bool first = true;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if ((h.flags >> e) & 1u) {
                const double v = first ? q[e] + cin : q[e];
                if (i < 0) *piece = v;
                else out[i] = v;
                first = false;
                ++i;
            }
        }
    } else {
#pragma unroll
        for (int m = 0; m < 4; ++m) *reinterpret_cast<double2 *>(lds + m * kQuarter + tid * 2) = make_double2(q[2 * m], q[2 * m + 1]);
        __syncthreads();
        const int nrows = h.hi - h.lo, g = lanes_per_row(nrows), sub = tid & (g - 1);
        const int64_t start = (int64_t)chunk * kChunk;
        int k0 = h.k0, k1 = h.k1;
        for (int base = 0; base < nrows; base += kTeam / g) {
            const int row = base + tid / g;
            if (base > 0) {
                k0 = k1 = 0;
                if (row < nrows) {
                    k0 = (int)(P.rowptr[h.lo + row] - start);
                    k1 = (int)(P.rowptr[h.lo + row + 1] - start);
                }
            }
            double t = 0.0;
            int k = k0 + sub;
            for (; k + 7 * g < k1; k += 8 * g) {   // eight reads on their way at a time
                double part[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) part[j] = lds[k + j * g];
#pragma unroll
                for (int j = 0; j < 8; ++j) t += part[j];
            }
            for (; k < k1; k += g) t += lds[k];
            t = group_sum(t, g);
            if (row < nrows && sub == 0) lds[kProdDoubles + row] = t;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void hand_over(uint64_t *place, double v) { __hip_atomic_store(place, (uint64_t)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void clear(uint64_t *place) { __hip_atomic_store(place, kEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// What a launch does: the whole solve, or of one step the rows that fit into a chunk, or those longer than a chunk behind a launch
// that did the others.
enum Part { PART_ALL, PART_CHUNKS, PART_LONG };

// One product, and what is done with every row's sum: aux = load(row) is asked for before the sum is known, apply(row, sum, aux)
// takes it.  h: the workgroup's first chunks, fetched already.  False: given up.
template <bool SEG, Part PART, class Load, class Apply>
__device__ __forceinline__ bool product(const ChunkPlan &P, Chunk &h, int how, const double *x, double beta, bool square, double *lds,
                                        double *piece, int *bad, GridBarrier &grid, int tid, const Load &load, const Apply &apply)
{
    const int team = __builtin_amdgcn_readfirstlane(threadIdx.x / kTeam), teams = blockDim.x / kTeam;
    const int per = (int)gridDim.x * teams;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int long0 = (int)blockIdx.x + (int)gridDim.x * wave;   // the first long row that this wavefront finishes
    int4 R = make_int4(0, 0, 0, 0);
    if (SEG && long0 < P.nlong) R = P.long_row[long0];
    Chunk next;
    for (int c0 = 0; PART != PART_LONG && c0 < P.nchunks; c0 += per) {
        const int chunk = c0 + team * (int)gridDim.x + (int)blockIdx.x;
        if (c0 > 0) {
            __syncthreads();   // the sums of the chunk before have been read
            h = next;
        }
        if (c0 + per < P.nchunks) load_chunk<SEG>(P, chunk + per, tid, next);
        int r = h.lo + tid;
        auto aux = load(r < h.hi ? r : 0);
        chunk_sums<SEG>(P, chunk, tid, h, how, x, beta, square, lds, piece);
        int skip = -1;
        if constexpr (SEG) {
            if (h.lr.x >= 0 || h.lr.y >= 0) {
                if (h.lr.y >= 0) skip = P.long_row[h.lr.y].x;
                if (tid >= kTeam - kWave) {   // the last wavefront hands the pieces of the long rows over
                    const bool one = tid == kTeam - kWave;
                    if (one && h.lr.x >= 0) hand_over(P.pieces + chunk, *piece);
                    if (one && h.lr.y >= 0) hand_over(P.pieces + P.nchunks + h.lr.y, lds[kOutOffset + h.tab.y - 1]);
                }
            }
        }
        int seg = h.seg;
        while (r < h.hi) {
            if (r != skip) {
                const double sum = SEG ? (seg >= 0 ? lds[kOutOffset + seg - h.tab.x] : 0.0) : lds[kProdDoubles + r - h.lo];
                apply(r, sum, aux);
            }
            r += kTeam;
            if (r >= h.hi) break;
            if constexpr (SEG) seg = P.row_seg[r];
            aux = load(r);
        }
    }
    if constexpr (SEG && PART != PART_CHUNKS) {
        if (P.nlong > 0) {
            for (int l = long0; l < P.nlong; l += (int)(gridDim.x * blockDim.x / kWave)) {
                if (l > long0) R = P.long_row[l];
                const auto aux = load(R.x);
                // lane k has the pieces k, k + 64, ...; the row's first one goes with the last of lane 0
                double z = 0.0;
                bool there = true;
                for (int k = lane; k <= R.z && there; k += kWave) there = grid.take(P.pieces + (k < R.z ? R.y + k : P.nchunks + l), kEmpty, z);
                if (__ballot(!there) != 0) {
                    if (lane == 0) *bad = 1;
                    break;
                }
                z = wave_sum(z);
                if (lane == 0) apply(R.x, z, aux);
            }
            __syncthreads();
            if (*bad) return false;
        }
    }
    return true;
}

// fn(row) for the rows that `product` hands to this workgroup
template <bool SEG, class F>
__device__ __forceinline__ void own_rows(const ChunkPlan &P, int tid, const F &fn)
{
    const int team = __builtin_amdgcn_readfirstlane(threadIdx.x / kTeam);
    for (int chunk = team * (int)gridDim.x + (int)blockIdx.x; chunk < P.nchunks; chunk += (int)(gridDim.x * blockDim.x / kTeam)) {
        const int lo = P.row_lo[chunk], hi = P.row_lo[chunk + 1];
        int skip = -1;
        if constexpr (SEG) {
            const int l = P.chunk_long[chunk].y;
            if (l >= 0) skip = P.long_row[l].x;
        }
        for (int r = lo + tid; r < hi; r += kTeam)
            if (r != skip) fn(r);
    }
    if constexpr (SEG) {
        if ((threadIdx.x & (kWave - 1)) != 0) return;
        for (int l = (int)blockIdx.x + (int)gridDim.x * (int)(threadIdx.x / kWave); l < P.nlong; l += (int)(gridDim.x * blockDim.x / kWave)) fn(P.long_row[l].x);
    }
}

// ------------------------------------------------------------------ what follows from the sums of a step (one thread of every workgroup)
__device__ __forceinline__ void finish(CsrState &S, int status)
{
    S.status = status;
    S.converged = status == TRON_OK;
    S.step = STEP_END;
}

// zz: z.z at the start, z = -g / M
__device__ __forceinline__ void begin_cg(CsrState &S, const CsrSolveArgs &A, double zz)
{
    S.rr = S.pMp = S.gscaled * S.gscaled;
    S.pp = zz;
    S.sMp = S.ss = 0.0;
    S.tol = A.xi * S.gscaled;
    S.it = 0;
    S.onb = 0;
    S.beta = 0.0;
    S.step = STEP_CG;
    if (sqrt(S.rr) <= S.tol) finish(S, TRON_EMAXITER);   // r.z has underflowed: no step to take
}

__device__ __forceinline__ void started(CsrState &S, const CsrSolveArgs &A)
{
    if (S.gnorm0 == 0.0) S.gnorm0 = S.gnorm;
    S.gscaled = S.delta = S.gnorm;
    if (S.gnorm <= A.eps * S.gnorm0) finish(S, TRON_OK);
    else if (A.blend > 0.0) {
        S.first_diag = 1;
        S.step = STEP_DIAG;
    } else begin_cg(S, A, S.gnorm * S.gnorm);
}

__device__ __forceinline__ void decide(CsrState &S, const CsrSolveArgs &A, const double (&t)[kSums], bool report)
{
    const double eta0 = 1e-4, eta1 = 0.25, eta2 = 0.75, sig2 = 0.5, sig3 = 4.0;
    const int step = S.step;
    S.turn = S.turn == 2 ? 0 : S.turn + 1;
    if (with_x(step)) S.na += 1;
    else if (step != STEP_ZERO_G) {
        S.pair_at = S.nb % kRing;
        S.nb += 1;
    }
    if (step == STEP_START) {
        S.ww = t[1];
        S.f = 0.5 * S.ww + A.C * t[0];
        S.step = STEP_START_G;
    } else if (step == STEP_START_G) {
        S.gnorm = sqrt(t[0]);
        S.n_fun = S.n_grad = 1;
        if (S.ww != 0.0) S.step = STEP_ZERO;   // the gradient at zero is the reference of the stopping test
        else started(S, A);
    } else if (step == STEP_ZERO) {
        S.step = STEP_ZERO_G;
    } else if (step == STEP_ZERO_G) {
        S.gnorm0 = sqrt(t[0]);
        S.n_fun += 1;
        S.n_grad += 1;
        started(S, A);
    } else if (step == STEP_DIAG) {
        S.gscaled = sqrt(t[0]);
        if (S.first_diag) S.delta = S.gscaled;
        S.first_diag = 0;
        begin_cg(S, A, t[1]);
    } else if (step == STEP_RESTART) {
        begin_cg(S, A, t[1]);
    } else if (step == STEP_CG) {
        // the step length, or the step to the boundary along p
        const double pHp = fma(A.C, t[0], S.pp), pp = S.pMp, sp = S.sMp, ss = S.ss;
        const double alpha = S.rr / pHp;
        S.length = alpha;
        if (sqrt(ss + alpha * (2.0 * sp + alpha * pp)) >= S.delta) {
            const double gap = S.delta * S.delta - ss;
            const double rad = sqrt(sp * sp + pp * gap);
            S.length = (sp >= 0.0) ? gap / (sp + rad) : (rad - sp) / pp;
            S.onb = 1;
        }
        S.step = STEP_HV;
    } else if (step == STEP_HV) {
        S.it += 1;
        S.n_hv += 1;
        S.cg_total += 1;
        const double rr = t[0];
        if (S.onb || S.it >= A.max_cg || sqrt(rr) <= S.tol) {
            S.pred = -0.5 * (t[1] - t[2]);
            S.snorm = sqrt(t[3]);
            S.ww = t[4];
            S.step = STEP_TRIAL;
        } else {
            // what the next step needs of p = z + beta p: p.p, and the M-weighted p.p, s.p, s.s (M z = r)
            const double beta = rr / S.rr, zz = A.blend > 0.0 ? t[7] : rr, zp = A.blend > 0.0 ? t[8] : t[5];
            S.beta = beta;
            S.rr = rr;
            S.pp = fma(beta, fma(beta, S.pp, 2.0 * zp), zz);
            S.pMp = fma(beta, fma(beta, S.pMp, 2.0 * t[5]), rr);
            S.sMp = fma(beta, t[6], t[2]);
            S.ss = t[3];
            S.step = STEP_CG;
        }
    } else if (step == STEP_TRIAL) {
        S.fnew = 0.5 * S.ww + A.C * t[0];
        S.step = STEP_TRIAL_G;
    } else {   // STEP_TRIAL_G
        S.n_fun += 1;
        const double ared = S.f - S.fnew;
        const bool noise = fabs(ared) <= 1e-12 * fabs(S.f) && S.pred <= 1e-12 * fabs(S.f);
        const double sigma = noise ? 1.0 : ared / S.pred;
        const double before = S.gnorm;
        if (sigma < eta1) S.delta = sig2 * fmin(S.snorm, S.delta);
        else if (sigma < eta2) { /* unchanged */ }
        else S.delta = fmin(sig3 * S.delta, fmax(S.delta, sig3 * S.snorm));
        const bool accepted = sigma > eta0;
        if (accepted) {
            S.cur ^= 1;
            S.dcur ^= 1;
            S.f = S.fnew;
            S.gnorm = S.gscaled = sqrt(t[0]);
            S.n_grad += 1;
        }
        S.outer += 1;
        if (S.trace_len < A.trace_cap) {
            if (report) {
                tron_trace_rec &q = S.trace_len < kHostRecords ? A.host->trace[S.trace_len] : A.trace[S.trace_len - kHostRecords];
                q.iter = S.outer; q.cg_iters = S.it; q.accepted = accepted ? 1 : 0; q.on_boundary = S.onb;
                q.f = S.f; q.gnorm = S.gnorm; q.delta = S.delta; q.ared = ared; q.pred = S.pred; q.snorm = S.snorm;
            }
            S.trace_len += 1;
        }
        if (accepted && S.gnorm <= A.eps * S.gnorm0) finish(S, TRON_OK);
        else if (S.pred <= 0.0 || (noise && S.gnorm >= before)) finish(S, TRON_EMAXITER);
        else if (S.outer >= A.max_outer) finish(S, TRON_EMAXITER);
        else if (!accepted) S.step = STEP_RESTART;
        else if (A.blend > 0.0) S.step = STEP_DIAG;
        else begin_cg(S, A, S.gnorm * S.gnorm);
    }
}

// to[k * stride] = the sum of v[k] over the wavefront, for the first n of them: two, seven or all nine.  Eight sums at a time are
// folded together, lane l ending with the sum of v[l mod 8]: ten additions instead of 48.
__device__ __forceinline__ void wave_sums(const double (&v)[kSums], int n, double *to, int stride)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (n <= 2) {
        double t = fold<0xB1>(v[0], v[1], lane & 1);
        t += dpp_move<0x4E>(t);
        t += other_quad_of_8(t);
        t += dpp_move<0x128>(t);   // lane ^ 8
        t = add_halves(add_row_pairs(t));
        if (lane < 2) to[lane * stride] = t;
        return;
    }
    double a[4], b[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = fold<0xB1>(v[2 * k], v[2 * k + 1], lane & 1);
#pragma unroll
    for (int k = 0; k < 2; ++k) b[k] = fold<0x4E>(a[2 * k], a[2 * k + 1], lane & 2);
    const double keep = (lane & 4) ? b[1] : b[0], give = (lane & 4) ? b[0] : b[1];
    double t = keep + other_quad_of_8(give);
    t += dpp_move<0x128>(t);
    t = add_halves(add_row_pairs(t));
    if (lane < 8) to[lane * stride] = t;
    if (n > 8) {
        const double last = wave_sum(v[8]);
        if (lane == 0) to[8 * stride] = last;
    }
}

// lane k has the grid's sum k, of what its workgroups (256 at most, a thread each) have left in `sums`: added up by the first team, the
// partial sums of its wavefronts behind a barrier in red
__device__ __forceinline__ void grid_sums(const double *sums, int nsums, int tid, double (*red)[kMaxTeams * kWavesPerBlock])
{
    double t[kSums];
    const bool mine = tid < (int)gridDim.x;
#pragma unroll
    for (int k = 0; k < kSums; ++k) t[k] = (k < nsums && mine) ? load_shared(sums + k * kMaxResidentGrid + tid) : 0.0;
    wave_sums(t, nsums, &red[0][tid / kWave], kMaxTeams * kWavesPerBlock);
}

__device__ __forceinline__ int sums_of(int step, bool precond) { return step != STEP_HV ? 2 : precond ? kSums : kSums - 2; }

// The first workgroup tells the host: the end of the solve, with the result, or (PART_ALL) that the solve goes on in another launch.
template <Part PART>
__device__ __forceinline__ void report_end(const CsrSolveArgs &A, const CsrState &S, int step)
{
    if (step == STEP_END && A.out) {
        const double *w = S.cur ? A.w[1] : A.w[0];
        for (int64_t j = threadIdx.x; j < A.d; j += blockDim.x) store_shared(A.out + j, load_shared(w + j));
    }
    // the host may go on when it sees the stamp: the result has arrived by then
    stores_arrived();
    __syncthreads();
    if (threadIdx.x == 0) {
        if (PART == PART_ALL) *A.state = S;
        A.host->st = S;
        __hip_atomic_store(&A.host->stamp, A.stamp, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// PART_ALL: the whole solve, as described at the top of the file.
// PART_CHUNKS and PART_LONG: a step in two launches (the second where there are rows longer than a chunk), for solves that find the GPU held
// by others: nothing waits inside, so that launches of several solves may share the GPU in any way.  Every workgroup has the
// same rows, and every sum is formed in the same order, as in the one launch, so the results have the same bits.  PART_CHUNKS begins with the
// sums of the step before and what follows from them; the state lies in one of two places in turn, as late workgroups may still
// be reading.  Where rows longer than a chunk follow, the wavefronts that will have them leave their lanes' shares of the sums in `lanes`, the
// others their sums in `waves`.
template <bool SEGX, bool SEGT, Part PART>
__global__ __launch_bounds__(kTeam * kMaxTeams) void k_csr_solve(ChunkPlan X, ChunkPlan T, CsrSolveArgs args)
{
    extern __shared__ __align__(16) double lds_all[];
    __shared__ CsrState S;
    __shared__ CsrSolveArgs A;
    __shared__ double red[kSums][kMaxTeams * kWavesPerBlock];
    __shared__ double pieces[kMaxTeams];
    __shared__ int bad;
    int tid = threadIdx.x & (kTeam - 1);
    const int team = __builtin_amdgcn_readfirstlane(threadIdx.x / kTeam);
    int first = team * (int)gridDim.x + (int)blockIdx.x;
    double *lds = lds_all + team * kTeamLds, *piece = pieces + team;
    GridBarrier grid(args.sync);
    if (threadIdx.x == 0) {
        bad = 0;
        A = args;
        if (args.resume) S = args.state[PART == PART_ALL ? 0 : PART == PART_LONG ? args.stamp & 1 : ~args.stamp & 1];
        else {
            S = CsrState{};
            S.turn = args.turn;
            S.step = STEP_START;
            S.status = TRON_EMAXITER;
        }
    }
    __syncthreads();
    const bool precond = A.blend > 0.0, report = blockIdx.x == 0, flat = PART == PART_ALL && gridDim.x <= kSyncFlat;
    int step = __builtin_amdgcn_readfirstlane(S.step), left = PART == PART_ALL ? A.steps : (int)(args.stamp & 1) + 1;   // its parity says which of the two places the sums go to
    if constexpr (PART == PART_CHUNKS) {
        if (args.resume && step != STEP_END) {
            const int nsums = sums_of(step, precond);
            if (team == 0) grid_sums(A.sums + (~left & 1) * kSums * kMaxResidentGrid, nsums, tid, red);
            __syncthreads();
            if (threadIdx.x < kWave) {
                const double *part = red[(int)threadIdx.x < nsums ? threadIdx.x : 0];
                const double total = (part[0] + part[1]) + (part[2] + part[3]);
                CsrState next = S;
                double t[kSums];
#pragma unroll
                for (int k = 0; k < kSums; ++k) t[k] = read_lane(total, k);
                decide(next, A, t, report && threadIdx.x == 0);
                if (threadIdx.x == 0) S = next;
            }
            __syncthreads();
            step = __builtin_amdgcn_readfirstlane(S.step);
            if (step == STEP_END && report) report_end<PART>(A, S, step);
        }
        if (report && threadIdx.x == 0) {
            A.state[args.stamp & 1] = S;
            if (step != STEP_END) __hip_atomic_store(&A.host->step, A.stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    // rows longer than a chunk in this step, and the first one of this wavefront
    int nlong = 0, long0 = 0;
    if constexpr (PART != PART_ALL) {
        nlong = step == STEP_RESTART ? 0 : with_x(step) ? (SEGX ? X.nlong : 0) : (SEGT ? T.nlong : 0);
        long0 = (int)blockIdx.x + (int)gridDim.x * __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
        if (PART == PART_LONG && nlong == 0) return;
    }
    Chunk h;
    if constexpr (PART != PART_LONG) {
        if (with_x(step)) load_chunk<SEGX>(X, first, tid, h);
        else load_chunk<SEGT>(T, first, tid, h);
    }
    bool ok = true;
    for (; step != STEP_END && left > 0; --left) {
        // as if they changed: the addresses of the first chunk are formed again instead of being kept through all steps
        if constexpr (PART == PART_ALL) asm volatile("" : "+v"(tid), "+s"(first));
        const int cur = __builtin_amdgcn_readfirstlane(S.cur), dcur = __builtin_amdgcn_readfirstlane(S.dcur);
        const bool fresh = __builtin_amdgcn_readfirstlane(S.it) == 0;
        const int pair_at = __builtin_amdgcn_readfirstlane(S.pair_at);
        const double *pair = A.pairs[pair_at], *point = A.point;
        const double *w = cur ? A.w[1] : A.w[0], *g = cur ? A.g[1] : A.g[0];
        const int na = __builtin_amdgcn_readfirstlane(S.na), nb = __builtin_amdgcn_readfirstlane(S.nb);
        double v[kSums] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        bool any = false;   // whether this lane had a row
        if constexpr (PART == PART_LONG) {
            if (long0 < nlong) {
                any = true;
#pragma unroll
                for (int k = 0; k < kSums; ++k)
                    if (k < sums_of(step, precond)) v[k] = A.lanes[((int64_t)long0 * kSums + k) * kWave + (threadIdx.x & (kWave - 1))];
            }
        }
        const int turn = __builtin_amdgcn_readfirstlane(S.turn);
        if (flat && threadIdx.x < kSums) clear(A.lines + ((turn == 2 ? 0 : turn + 1) * kSyncFlat + blockIdx.x) * kLine + threadIdx.x);
        if (with_x(step)) {
            const bool cg = step == STEP_CG, lr = A.loss == TRON_LOSS_LR;
            double *u = A.u[na % kRing];
            double *D = (dcur ^ (step == STEP_ZERO || step == STEP_TRIAL)) ? A.D[1] : A.D[0];
            const double *row_in = cg ? D : A.y;
            const double beta = S.beta;
            ok = product<SEGX, PART>(X, h, cg ? GATHER_PAIR : step == STEP_ZERO ? GATHER_NONE : GATHER_ONE, cg ? pair : step == STEP_START ? A.w0 : point, beta, false,
                               lds, piece, &bad, grid, tid, [&](int r) { return row_in[r]; },
                               [&](int r, double z, double in) {
                                   any = true;
                                   double t;
                                   if (cg) {
                                       t = in * z;
                                       v[0] = fma(z, t, v[0]);
                                   } else {
                                       const RowTerms q = lr ? row_terms<TRON_LOSS_LR>(z, in) : row_terms<TRON_LOSS_L2SVM>(z, in);
                                       t = q.zhat;
                                       store_shared(D + r, q.D);
                                       v[0] += q.alpha;
                                   }
                                   store_shared(u + r, t);
                               });
            if (PART != PART_LONG && step == STEP_START)
                own_rows<SEGT>(T, tid, [&](int j) {
                    any = true;
                    const double x = A.w0[j];
                    store_shared(A.w[0] + j, x);
                    v[1] = fma(x, x, v[1]);
                });
        } else {
            const double *u = step == STEP_DIAG ? (dcur ? A.D[1] : A.D[0]) : A.u[(na + kRing - 1) % kRing];
            double *pair_out = A.pairs[nb % kRing], *point_out = A.point;
            if (PART != PART_LONG && step == STEP_RESTART) {
                own_rows<SEGT>(T, tid, [&](int j) {
                    any = true;
                    const double z = -g[j] / (precond ? A.M[j] : 1.0);
                    v[1] = fma(z, z, v[1]);
                    store_shared(pair_out + 2 * (int64_t)j, z);
                    store_shared(pair_out + 2 * (int64_t)j + 1, 0.0);
                });
            } else {
                const bool hv = step == STEP_HV, diag = step == STEP_DIAG, trial = step == STEP_TRIAL_G, zero = step == STEP_ZERO_G;
                const double length = S.length, beta = S.beta;
                double *gnew = (trial && cur == 0) ? A.g[1] : A.g[0], *wnew = cur ? A.w[0] : A.w[1];
                const double *wj = trial ? point : w;
                struct Aux { double w, g, p, s, r, m; };
                ok = product<SEGT, PART>(T, h, GATHER_ONE, u, 0.0, diag, lds, piece, &bad, grid, tid,
                                   [&](int j) {
                                       Aux a{zero ? 0.0 : wj[j], 0.0, 0.0, 0.0, 0.0, 1.0};
                                       if (hv || diag) a.g = g[j];
                                       if (hv) {
                                           const v2d q = reinterpret_cast<const v2d *>(pair)[j];
                                           a.p = fma(beta, q.y, q.x);
                                           a.s = A.s[j];
                                           a.r = A.r[j];
                                           if (precond) a.m = A.M[j];
                                       }
                                       return a;
                                   },
                                   [&](int j, double z, const Aux &a) {
                                       any = true;
                                       double first, second = 0.0;   // the pair to gather from next
                                       if (hv) {
                                           const double Hp = fma(A.C, z, a.p);
                                           const double s = fma(length, a.p, fresh ? 0.0 : a.s), r = fma(-length, Hp, fresh ? -a.g : a.r), x = a.w + s;
                                           first = r / a.m;
                                           second = a.p;
                                           A.s[j] = s;
                                           A.r[j] = r;
                                           store_shared(point_out + j, x);
                                           v[0] = fma(r, first, v[0]);
                                           v[1] = fma(a.g, s, v[1]);
                                           v[2] = fma(s, r, v[2]);
                                           v[3] = fma(a.m * s, s, v[3]);
                                           v[4] = fma(x, x, v[4]);
                                           v[5] = fma(r, a.p, v[5]);
                                           v[6] = fma(a.m * s, a.p, v[6]);
                                           v[7] = fma(first, first, v[7]);
                                           v[8] = fma(first, a.p, v[8]);
                                       } else if (diag) {
                                           const double m = fma(A.blend * A.C, z, 1.0);
                                           first = -a.g / m;
                                           A.M[j] = m;
                                           v[0] = fma(-a.g, first, v[0]);
                                           v[1] = fma(first, first, v[1]);
                                       } else {
                                           const double o = fma(A.C, z, a.w);
                                           v[0] = fma(o, o, v[0]);
                                           if (zero) return;
                                           first = -o;
                                           gnew[j] = o;
                                           if (trial) store_shared(wnew + j, a.w);
                                       }
                                       store_shared(pair_out + 2 * (int64_t)j, first);
                                       store_shared(pair_out + 2 * (int64_t)j + 1, second);
                                   });
            }
        }
        const int used = with_x(step) ? na : nb;   // how many places were used before this step's
        if (!ok) break;
        // the workgroup's sums
        const int nsums = sums_of(step, precond);
        double *sums = A.sums + (left & 1) * kSums * kMaxResidentGrid;
        if (PART == PART_CHUNKS && long0 < nlong) {
#pragma unroll
            for (int k = 0; k < kSums; ++k)
                if (k < nsums) A.lanes[((int64_t)long0 * kSums + k) * kWave + (threadIdx.x & (kWave - 1))] = v[k];
        } else if (PART == PART_LONG && long0 >= nlong) {
            if ((int)(threadIdx.x & (kWave - 1)) < nsums)
                red[threadIdx.x & (kWave - 1)][threadIdx.x / kWave] = A.waves[((int64_t)blockIdx.x * kSums + (threadIdx.x & (kWave - 1))) * kMaxTeams * kWavesPerBlock + threadIdx.x / kWave];
        } else if (__ballot(any)) wave_sums(v, nsums, &red[0][threadIdx.x / kWave], kMaxTeams * kWavesPerBlock);
        else if ((int)(threadIdx.x & (kWave - 1)) < nsums) red[threadIdx.x & (kWave - 1)][threadIdx.x / kWave] = 0.0;
        // Up to 64 workgroups need no barrier beside the sums: each waits until those of all are there, a lane for every workgroup.  (The
        // lines of the next turn were cleared before; all have read what was in them, or they would not have got here.)
        if (flat) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // what the others read has arrived
        __syncthreads();
        if (PART == PART_CHUNKS && nlong > 0) {
            if ((int)threadIdx.x < nsums * kMaxTeams * kWavesPerBlock)   // (those of the wavefronts that have left their lanes' are not read)
                A.waves[(int64_t)blockIdx.x * kSums * kMaxTeams * kWavesPerBlock + threadIdx.x] = (&red[0][0])[threadIdx.x];
            return;
        }
        if ((int)threadIdx.x < nsums) {
            double part[kMaxTeams * kWavesPerBlock], t = 0.0;
#pragma unroll
            for (int k = 0; k < kMaxTeams * kWavesPerBlock; ++k) part[k] = red[threadIdx.x][k];
#pragma unroll
            for (int k = 0; k < kMaxTeams * kWavesPerBlock; ++k)
                if (k < (int)blockDim.x / kWave) t += part[k];
            if (flat) hand_over(A.lines + (turn * kSyncFlat + blockIdx.x) * kLine + threadIdx.x, t);
            else store_shared(sums + threadIdx.x * kMaxResidentGrid + blockIdx.x, t);
        }
        if (PART != PART_ALL) return;
        if (!flat) grid.arrive();
        // most often a product with the other orientation follows
        if (with_x(step)) load_chunk<SEGT>(T, first, tid, h);
        else load_chunk<SEGX>(X, first, tid, h);
        if (!flat) {
            ok = grid.wait();
            if (!ok) break;
            if (team == 0) grid_sums(sums, nsums, tid, red);
            __syncthreads();
        }
        if (threadIdx.x < kWave) {   // all of the wavefront the same; lane k has sum k
            double total;
            if (flat) {
                double t[kSums];
                ok = grid.collect(A.lines + (turn * kSyncFlat + threadIdx.x) * kLine, nsums, kEmpty, t);
                wave_sums(t, nsums, &red[0][0], kMaxTeams * kWavesPerBlock);
                total = red[(int)threadIdx.x < nsums ? threadIdx.x : 0][0];
                if (!ok && threadIdx.x == 0) bad = 1;
            } else {
                const double *part = red[(int)threadIdx.x < nsums ? threadIdx.x : 0];
                total = (part[0] + part[1]) + (part[2] + part[3]);
            }
            if (used >= kRing && used % kRing == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the places are used again
            CsrState next = S;
            double t[kSums];
#pragma unroll
            for (int k = 0; k < kSums; ++k) t[k] = read_lane(total, k);
            decide(next, A, t, report && threadIdx.x == 0);
            if (threadIdx.x == 0) S = next;
        }
        __syncthreads();
        ok = bad == 0;
        if (!ok) break;
        const bool was_x = with_x(step);
        step = __builtin_amdgcn_readfirstlane(S.step);
        if (step == STEP_DIAG || step == STEP_TRIAL) {   // they gather from D and the trial point, which lie in the same places every time
            if (threadIdx.x < kWave) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __syncthreads();
        }
        if (!was_x && !with_x(step) && step != STEP_END) load_chunk<SEGT>(T, first, tid, h);   // DIAG, RESTART after a gradient
        // (RESTART and DIAG are followed by a product with X, fetched during the wait like after every other step with X^T)
    }
    if (PART != PART_ALL) return;
    if (ok && report) report_end<PART>(A, S, step);
    grid.leave();
}

// ------------------------------------------------------------------ host
// The work space of a handle's solves, kept with the handle: 16 d + 4 n doubles and a little
constexpr int kPieces = 2 * kRing + 9;
struct CsrSolver {
    double *blocks[kPieces];     // what was allocated
    int nblocks = 0;
    bool ready = false;
    CsrHost *host = nullptr, *host_dev = nullptr;
    tron_trace_rec *trace = nullptr;   // device memory, records past the first kHostRecords
    int trace_cap = 0;
    bool lds_set[3] = {false, false, false};   // by Part
    int64_t to_clear = 0;        // places from args.lines on that are kEmpty between solves,
    bool cleared = false;        // unless one was given up (or none was made yet); of the lines, those of the turn `turn`
    int turn = 0;
    double *step_block = nullptr;   // what launches per step need beside it
    int64_t steps = 0;           // such launches so far
    ChunkPlan X, T;
    CsrSolveArgs args;
};

static void csr_resident_free(CsrSolver &W)
{
    for (int k = 0; k < W.nblocks; ++k) hipFree(W.blocks[k]);
    W.nblocks = 0;
}

void csr_resident_release(tron_dataset *ds)
{
    if (!ds->csr_solver) return;
    csr_resident_free(*ds->csr_solver);
    hipFree(ds->csr_solver->trace);
    hipFree(ds->csr_solver->step_block);
    delete ds->csr_solver;
    ds->csr_solver = nullptr;
}

__global__ __launch_bounds__(kBlock) void k_clear(uint64_t *places, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) places[i] = kEmpty;
}

// Layouts of large matrices (several column ranges, values left out) stay with a launch per product, whose workgroups keep four times
// as many wavefronts on a compute unit: the more rounds of chunks, the less there is to gain.  us a solve (a handle's first one), driven by
// the host / in one launch, Zipf-distributed columns: 623 chunks 998 / 888 (1026 / 936), 1064 1286 / 1087 (1339 / 1167), 1402 1568 / 1252,
// 1712 1623 / 1441 (1739 / 1549), 2146 1957 / 1798 (2064 / 1954); uniform ones: 2283 524 / 503 (614 / 587), 2420 483 / 417 (584 / 527).  Rows longer than a
// chunk among the plain layout's, which a launch of their own completes, and chunks of so many rows that the threads would go over
// them one after the other are left to the host, too.
constexpr int kMaxRounds = 5;

static bool plan_fits(const CsrPlan &A)
{
    if (A.P != 1 || A.unit || A.cols >= (1 << 28)) return false;
    return A.plain ? A.nfix == 0 && A.max_rows <= kPlainRows : A.direct && A.max_rows <= kSegRows;
}

static ChunkPlan chunk_plan(const CsrPlan &A)
{
    return ChunkPlan{A.col, A.val, A.row_lo, A.rowptr, A.chunk_tab, A.flags, A.row_seg, A.chunk_long, A.long_row, nullptr, A.part_nnz[0], A.nblocks, A.plain ? 0 : A.nfix};
}

struct Piece {
    double **p;
    int64_t size;   // doubles
};

// Up to 2 MB an allocation comes from memory that the runtime has at hand or fetches 2 MB at a time (1 to 40 us), a larger one takes 25 to
// 500 us each time: the pieces share blocks of up to 2 MB, and where one of them is larger (pairs of more than 131,072 columns) one block.
// First solve of a handle with 20,000 rows in us (means; single ones differ by 200), an allocation a piece / this / driven by the host: 110,000
// columns 610 / 580 / 580, 160,000 1130 / 640 / 730, 200,000 1170 / 690 / 690, 300,000 1970 / 730 / 1500 (and freeing them 1290 / 490 / 540).
static int allocate(CsrSolver &W, const Piece *pieces, int count)
{
    constexpr int64_t kSmall = (2 << 20) / sizeof(double), kAlign = 256 / sizeof(double);
    auto rounded = [&](int k) { return (pieces[k].size + kAlign - 1) / kAlign * kAlign; };
    int64_t largest = 0;
    for (int k = 0; k < count; ++k) largest = std::max(largest, rounded(k));
    csr_resident_free(W);
    for (int k0 = 0, k1 = 0; k0 < count; k0 = k1) {
        int64_t total = 0;
        for (; k1 < count && (k1 == k0 || largest > kSmall || total + rounded(k1) <= kSmall); ++k1) total += rounded(k1);
        double *block = nullptr;
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&block), sizeof(double) * total));
        W.blocks[W.nblocks++] = block;
        for (int k = k0; k < k1; block += rounded(k), ++k) *pieces[k].p = block;
    }
    return TRON_OK;
}

static int ensure_space(tron_dataset *ds, int trace_cap)
{
    if (!ds->csr_solver) {
        ds->csr_solver = new (std::nothrow) CsrSolver();
        if (!ds->csr_solver) { set_error("out of host memory"); return TRON_ENOMEM; }
    }
    CsrSolver &W = *ds->csr_solver;
    CsrSolveArgs &A = W.args;
    if (!W.ready) {
        const int64_t px = ds->fwd.plain || !ds->fwd.nfix ? 0 : ds->fwd.nblocks + ds->fwd.nfix, pt = ds->bwd.plain || !ds->bwd.nfix ? 0 : ds->bwd.nblocks + ds->bwd.nfix;
        const int64_t psums = 2 * kSums * kMaxResidentGrid, pstate = (sizeof(CsrState) + 7) / 8 / kLine * kLine + kLine, lines = 3 * kSyncFlat * kLine;
        Piece pieces[kPieces];
        int m = 0;
        for (int k = 0; k < kRing; ++k) pieces[m++] = Piece{&A.pairs[k], 2 * ds->d};
        for (int k = 0; k < kRing; ++k) pieces[m++] = Piece{&A.u[k], ds->n};
        for (double **v : {&A.point, &A.w[0], &A.w[1], &A.g[0], &A.g[1], &A.s, &A.r, &A.M}) pieces[m++] = Piece{v, ds->d};
        pieces[m++] = Piece{&A.sums, psums + pstate + lines + px + pt};
        TRON_TRY(allocate(W, pieces, m));
        A.state = reinterpret_cast<CsrState *>(A.sums + psums);
        W.X = chunk_plan(ds->fwd);
        W.T = chunk_plan(ds->bwd);
        A.lines = reinterpret_cast<uint64_t *>(A.sums + psums + pstate);
        W.X.pieces = A.lines + lines;
        W.T.pieces = W.X.pieces + px;
        W.to_clear = lines + px + pt;
        A.n = ds->n;
        A.d = ds->d;
        A.y = ds->y;
        A.D[0] = ds->Dbuf[0];
        A.D[1] = ds->Dbuf[1];
        static_assert(sizeof(CsrHost) <= kSolveHostBytes, "room behind the scalars");
        W.host = reinterpret_cast<CsrHost *>(ds->scal_host + kHostWords);
        W.host_dev = reinterpret_cast<CsrHost *>(ds->scal_dev + kHostWords);
        W.host->step = W.steps;
        W.ready = true;
        W.cleared = false;
    }
    if (!W.cleared) {
        hipLaunchKernelGGL(k_clear, dim3((unsigned)((W.to_clear + kBlock - 1) / kBlock)), dim3(kBlock), 0, ds->stream, A.lines, W.to_clear);
        TRON_HIP(hipGetLastError());
        W.cleared = true;
    }
    if (trace_cap - kHostRecords > W.trace_cap) {
        TRON_HIP(hipFree(W.trace));
        W.trace = nullptr;
        W.trace_cap = 0;
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&W.trace), sizeof(tron_trace_rec) * (size_t)(trace_cap - kHostRecords)));
        W.trace_cap = trace_cap - kHostRecords;
    }
    return TRON_OK;
}

template <bool SEGX, bool SEGT, Part PART>
static int launch(tron_dataset *ds, CsrSolver &W, const CsrSolveArgs &A, int grid, int teams)
{
    const int lds = teams * kTeamLds * (int)sizeof(double);
    if (lds > 64 << 10 && !W.lds_set[PART]) TRON_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_csr_solve<SEGX, SEGT, PART>), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    W.lds_set[PART] = true;
    hipLaunchKernelGGL((k_csr_solve<SEGX, SEGT, PART>), dim3(grid), dim3(teams * kTeam), lds, ds->stream, W.X, W.T, A);
    TRON_HIP(hipGetLastError());
    return TRON_OK;
}

template <Part PART>
static int launch_part(tron_dataset *ds, CsrSolver &W, const CsrSolveArgs &A, int grid, int teams)
{
    return (ds->fwd.plain ? (ds->bwd.plain ? launch<false, false, PART> : launch<false, true, PART>) : (ds->bwd.plain ? launch<true, false, PART> : launch<true, true, PART>))(ds, W, A, grid, teams);
}

// The solve in one launch, or in several of kStepsPerLaunch steps: 1 = done, 0 = workgroups gave up waiting for others (w0 is as it was)
static int solve_resident(tron_dataset *ds, CsrSolver &W, CsrSolveArgs &A, int grid, int teams)
{
    for (int64_t stamp = 1;; ++stamp) {
        A.stamp = stamp;
        A.resume = stamp > 1;
        TRON_TRY(launch_part<PART_ALL>(ds, W, A, grid, teams));
        // With the stamp everything is there that the call returns (the stream's own wait takes some microseconds more)
        auto ended = [&]() { return __atomic_load_n(&W.host->stamp, __ATOMIC_ACQUIRE) == stamp; };
        for (unsigned spins = 1; !ended(); ++spins) {
            if ((spins & kSpinsPerQuery) == 0 && hipStreamQuery(ds->stream) != hipErrorNotReady) break;
            __builtin_ia32_pause();
        }
        if (!ended()) {
            (void)hipGetLastError();
            TRON_HIP(hipStreamSynchronize(ds->stream));
            if (!ended()) {
                W.cleared = false;
                return 0;
            }
        }
        if (W.host->st.step == STEP_END) break;
    }
    W.turn = W.host->st.turn;
    return 1;
}

// The same solve with a launch or two per step, for solves that do not wait for their turn (ResidentShare): kAhead steps enqueued behind the one that the host has seen begin
static int solve_in_steps(tron_dataset *ds, CsrSolver &W, CsrSolveArgs &A, int grid, int teams)
{
    constexpr int64_t kAhead = 3;
    const int nlong = std::max(W.X.nlong, W.T.nlong);
    if (!W.step_block) {
        const int64_t states = (2 * sizeof(CsrState) + 7) / 8, waves = (int64_t)kMaxResidentGrid * kSums * kMaxTeams * kWavesPerBlock;
        const int64_t lanes = (int64_t)std::min(nlong, kMaxResidentGrid * kMaxTeams * kWavesPerBlock) * kSums * kWave;
        TRON_HIP(hipMalloc(reinterpret_cast<void **>(&W.step_block), sizeof(double) * (waves + lanes + states)));
    }
    A.waves = W.step_block;
    A.lanes = A.waves + (int64_t)kMaxResidentGrid * kSums * kMaxTeams * kWavesPerBlock;
    A.state = reinterpret_cast<CsrState *>(A.lanes + (int64_t)std::min(nlong, kMaxResidentGrid * kMaxTeams * kWavesPerBlock) * kSums * kWave);
    A.sync.ticks = std::max<long long>(A.sync.ticks, 0);   // (the pieces of a long row are there: nothing is waited for)
    const int64_t before = W.steps;
    A.resume = 0;
    for (unsigned spins = 0;;) {
        if (__atomic_load_n(&W.host->stamp, __ATOMIC_ACQUIRE) != 0) return 1;
        const int64_t seen = std::max(__atomic_load_n(&W.host->step, __ATOMIC_ACQUIRE), before);
        if (W.steps <= seen + kAhead) {
            A.stamp = ++W.steps;
            TRON_TRY(launch_part<PART_CHUNKS>(ds, W, A, grid, teams));
            A.resume = 1;
            if (nlong > 0) TRON_TRY(launch_part<PART_LONG>(ds, W, A, grid, teams));
            spins = 0;
            continue;
        }
        if ((++spins & 1023u) != 0) { __builtin_ia32_pause(); continue; }
        // nothing for a while: make sure that the kernels are still running
        const hipError_t e = hipStreamQuery(ds->stream);
        (void)hipGetLastError();
        if (e != hipSuccess && e != hipErrorNotReady) return hip_fail(e, "hipStreamQuery", __FILE__, __LINE__);
        if (e == hipSuccess && __atomic_load_n(&W.host->stamp, __ATOMIC_ACQUIRE) == 0 && __atomic_load_n(&W.host->step, __ATOMIC_ACQUIRE) < W.steps) {
            set_error("internal: a step of a solve has ended without its word");
            return TRON_ESTATE;
        }
        std::this_thread::yield();
    }
}

int csr_resident_solve(tron_dataset *ds, const tron_params &Q, double *w_dev, tron_result *res, int *status)
{
    if (ds->prof.on || !plan_fits(ds->fwd) || !plan_fits(ds->bwd)) return 0;   // (the profiler times the kernels of the general path)
    const int most = std::max(ds->fwd.nblocks, ds->bwd.nblocks);
    const int cus = std::min(ds->cus, kMaxResidentGrid), grid = std::min(most, cus);
    const int teams = std::min(kMaxTeams, (most + grid - 1) / grid);
    if (most > kMaxRounds * grid * teams || !resident_possible(ds, grid)) return 0;
    const int cap = std::min(res->trace_cap, Q.max_outer);
    if (cap > kMaxRecords) return 0;
    // Where one launch is not to be tried, or is given up, the steps are launches of their own: the same bits.  (Without any wait, or without
    // room for the work space, the host drives the solve.)
    const bool one = ds->resident.try_it(g_tuning.solve_wait_us), steps = g_tuning.solve_wait_us != 0 || g_tuning.solve_resident > 0;
    if (!one && (!steps || ds->resident.no_room)) return 0;
    int rc = ensure_space(ds, cap);
    ds->resident.no_room = rc == TRON_ENOMEM;
    if (rc == TRON_ENOMEM) {   // the host-driven solve needs less
        (void)hipGetLastError();
        csr_resident_release(ds);
        ds->resident.ended(false);
        return 0;
    }
    if (rc != TRON_OK) return rc;
    CsrSolver &W = *ds->csr_solver;
    CsrSolveArgs A = W.args;
    A.w0 = w_dev;
    A.out = ds->d <= kOutInKernel ? w_dev : nullptr;
    A.loss = Q.loss;
    A.max_outer = Q.max_outer;
    A.max_cg = Q.max_cg;
    A.trace_cap = cap;
    A.C = Q.C;
    A.eps = Q.eps;
    A.xi = Q.cg_xi;
    A.blend = Q.precond_blend;
    A.sync = grid_sync(ds);
    A.host = W.host_dev;
    A.trace = W.trace;
    A.turn = W.turn;
    A.steps = kStepsPerLaunch;
    ds->have_D = false;
    {
        ResidentShare share(ds, grid, one ? (most <= grid * teams ? 1 : 2) : 0);
        W.host->stamp = 0;
        rc = 0;
        if (share.granted()) {
            rc = solve_resident(ds, W, A, grid, teams);
            if (rc < 0) return rc;
            ds->resident.ended(rc > 0);
            share.give_back();
        }
        if (rc == 0) {
            if (!steps) return 0;
            TRON_TRY(ensure_space(ds, cap));   // (places of a solve that was given up are cleared)
            rc = solve_in_steps(ds, W, A, grid, teams);
            if (rc == TRON_ENOMEM) {
                (void)hipGetLastError();
                return 0;
            }
            if (rc < 0) return rc;
        }
    }
    const CsrState &S = W.host->st;
    if (!A.out) {
        TRON_HIP(hipMemcpyAsync(w_dev, A.w[S.cur], sizeof(double) * ds->d, hipMemcpyDeviceToDevice, ds->stream));
        TRON_HIP(hipStreamSynchronize(ds->stream));
    }
    res->f = S.f;
    res->gnorm = S.gnorm;
    res->gnorm0 = S.gnorm0;
    res->outer_iters = S.outer;
    res->cg_iters_total = S.cg_total;
    res->n_fun = S.n_fun;
    res->n_grad = S.n_grad;
    res->n_hv = S.n_hv;
    res->converged = S.converged;
    res->trace_len = S.trace_len;
    for (int k = 0; k < std::min(S.trace_len, kHostRecords); ++k) res->trace[k] = W.host->trace[k];
    if (S.trace_len > kHostRecords) {
        TRON_HIP(hipStreamSynchronize(ds->stream));
        TRON_HIP(hipMemcpy(res->trace + kHostRecords, W.trace, sizeof(tron_trace_rec) * (size_t)(S.trace_len - kHostRecords), hipMemcpyDeviceToHost));
    }
    ds->Dcur = S.dcur;
    ds->have_D = true;
    *status = S.status;
    return 1;
}

}  // namespace tron
