// Register tile of the dense row-major kernels: how a wavefront covers rows and columns of X.
#pragma once

#include "device_util.h"

namespace tron {

// A wave tile of RT = U * 64 / L rows.  A row is covered by L consecutive lanes; lane q of them holds the columns
// col(q, 0) .. col(q, E - 1): pieces of one or two columns (8 or 16 bytes) dealt to the L lanes in turn, so that one
// load instruction reads L consecutive pieces of a row and the next one the pieces behind them.  (With E consecutive columns
// per lane every instruction touches all cache lines of its rows and takes a part of each: a Hessian-vector pass over
// 200,003 x 257 took 82 us, this way 70 us; 3M x 25 173 us against 158 us a call.)  Step u covers the 64 / L consecutive
// rows u * RW + lane / L; steps of rows that lie U apart, which would make lane i the owner of row i, took 192 us
// against 162 us on 5M x 18.  The sum over a row's lanes is folded so that step u's total ends up in the lanes with
// lane % U == u (row_sum), which own the row: no exchange through LDS between the sums, the per-row work and the way back.
// Staging whole tiles through LDS, 16 bytes per lane in memory order, was measured too: 227 us on 5M x 18, since the room
// for the tiles leaves two wavefronts per SIMD.
template <int E, int L, int U, bool VEC>
struct Tile {
    static constexpr int RW = kWave / L;     // rows per step
    static constexpr int RT = U * RW;        // rows per wave tile
    static_assert(U == (L < 4 ? L : 4), "row_sum folds the rows of a step over lanes of one quad");

    // column of entry e of lane q of a row
    __device__ static __forceinline__ constexpr int col(int q, int e) { return VEC ? (e / 2) * 2 * L + 2 * q + (e & 1) : e * L + q; }
    // the tile row a lane owns, and whether it is the first of the lanes that own it (L > 4: every quad of a row's lanes
    // owns the same U rows)
    __device__ static __forceinline__ int own_row(int lane) { return (lane % U) * RW + lane / L; }
    __device__ static __forceinline__ bool first_owner(int lane) { return lane % L < U; }

    // bit i of the result = the owner of tile row i passes true (tiles of 64 rows)
    __device__ static __forceinline__ uint64_t ballot_rows(bool pred, int lane)
    {
        static_assert(RT <= kWave, "");
        if constexpr (U == 1) return __ballot(pred);
        return __ballot(__shfl((int)pred, (lane % RW) * L + lane / RW, kWave) != 0);
    }

    // load the U x E block of this lane; out-of-range rows / columns read as zero.  rows: bit i clear = row row0 + i
    // is not needed (its coefficient is zero) and is not read at all
    __device__ static __forceinline__ void load(const double *__restrict__ X, int64_t n, int64_t d, int64_t row0,
                                                int lane, double (&x)[U][E], uint64_t rows = ~0ull)
    {
        const int q = lane % L, rl = lane / L;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t row = row0 + u * RW + rl;
            const bool rok = row < n && ((rows >> (u * RW + rl)) & 1u);
            const double *p = X + row * d;
            if (VEC) {
#pragma unroll
                for (int e = 0; e < E; e += 2) {
                    double2 t = make_double2(0.0, 0.0);
                    if (rok && col(q, e) < d) t = *reinterpret_cast<const double2 *>(p + col(q, e));
                    x[u][e] = t.x;
                    x[u][e + 1] = t.y;
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) x[u][e] = (rok && col(q, e) < d) ? p[col(q, e)] : 0.0;
            }
        }
    }

    // from each lane's partial sums of the U rows to the sum of the row this lane owns.  The first two steps over the row's
    // lanes fold the U rows into one value per lane; the remaining ones add the same lane of the other quads, in an order
    // that gives every owner of a row the same bits.
    __device__ static __forceinline__ double fold_rows(const double (&t)[U], int lane)
    {
        double s = t[0];
        if constexpr (U == 2) s = fold<0xB1>(t[0], t[1], lane & 1);
        if constexpr (U == 4) s = fold<0x4E>(fold<0xB1>(t[0], t[1], lane & 1), fold<0xB1>(t[2], t[3], lane & 1), lane & 2);
        if constexpr (L == 8) s += other_quad_of_8(s);
        if constexpr (L >= 16) {
            s += dpp_move<0x128>(s);   // row_ror:8 before row_ror:4: (q0 + q2) + (q1 + q3) in every quad
            s += dpp_move<0x124>(s);
        }
        if constexpr (L >= 32) s = add_row_pairs(s);
        if constexpr (L >= 64) s = add_halves(s);
        return s;
    }

    // x_row . vec for the row this lane owns
    __device__ static __forceinline__ double row_sum(const double (&x)[U][E], const double (&vec)[E], int lane)
    {
        double t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            t[u] = 0.0;
#pragma unroll
            for (int e = 0; e < E; ++e) t[u] = fma(x[u][e], vec[e], t[u]);
        }
        return fold_rows(t, lane);
    }

    // every lane receives, for step u, the value held by the owner of its row
    __device__ static __forceinline__ void from_row_owner(double mine, double (&c)[U])
    {
        if constexpr (U == 1) c[0] = mine;
        if constexpr (U == 2) { c[0] = dpp_move<0xA0>(mine); c[1] = dpp_move<0xF5>(mine); }   // quad_perm [0,0,2,2], [1,1,3,3]
        if constexpr (U == 4) { c[0] = dpp_move<0x00>(mine); c[1] = dpp_move<0x55>(mine); c[2] = dpp_move<0xAA>(mine); c[3] = dpp_move<0xFF>(mine); }
    }

    // acc[e] summed over the lanes that hold the same columns, then over the workgroup's wavefronts (`waves` of them):
    // column c goes to out[c * stride].  lds: waves * E * L doubles that nothing else uses any more.
    __device__ static __forceinline__ void flush(double (&acc)[E], int64_t d, int lane, int wv, int waves, double *lds,
                                                 double *__restrict__ out, int64_t stride)
    {
#pragma unroll
        for (int e = 0; e < E; ++e) {
#pragma unroll
            for (int m = L; m < kWave; m <<= 1) acc[e] += __shfl_xor(acc[e], m, kWave);
        }
        if (lane < L) {
#pragma unroll
            for (int e = 0; e < E; ++e) lds[wv * (E * L) + col(lane, e)] = acc[e];
        }
        __syncthreads();
        for (int c = threadIdx.x; c < d; c += waves * kWave) {
            double s = 0.0;
            for (int k = 0; k < waves; ++k) s += lds[k * (E * L) + c];
            store_shared(out + c * stride, s);
        }
    }
};

struct Shape { int E, L; };

// smallest L in {1,2,4,...,64} with E = ceil(d/L) <= 8; for even d an odd E is rounded up, so that every lane can
// use 16-byte loads (the columns past d are masked: d = 18 runs as 4 lanes x 3 pairs of columns, d = 28 as 4 x 4)
inline bool pick_shape(int64_t d, Shape &s)
{
    for (int L = 1; L <= kWave; L *= 2) {
        int64_t E = (d + L - 1) / L;
        if (E <= 8) {
            if (L > 1 && d % 2 == 0 && E % 2 == 1) E += 1;
            s.E = (int)E;
            s.L = L;
            return true;
        }
    }
    return false;
}

constexpr int pick_U(int E, int L) { return (L < 4 ? L : 4); }

}  // namespace tron
