// Register tile of the dense row-major kernels: how a wavefront covers rows and columns of X.
#pragma once

#include "device_util.h"

namespace tron {

typedef double v2d __attribute__((ext_vector_type(2)));

// Matrices that do not fit the 256 MB cache in front of HBM are read with non-temporal loads, at 7.0 instead of 6.2 TB/s; a smaller one gains
// nothing by it (TB/s of a plain sum over tiles of 12 KiB, ordinary / non-temporal loads: 192 MB 6.4 / 6.4, 256 MB 6.7 / 6.6, 288 MB 6.5 / 6.7, 512 MB
// 6.0 / 6.9, 2 GB 6.2 / 7.0, 8 GB 6.3 / 7.1), but then a line must be fetched by one instruction as a whole: where an instruction reads pieces of 64 bytes of
// rows, the same loads lose a quarter (2 GB of rows of 24: 5.5 / 4.8).  So
//   - rows of 9 to 32 columns (two and four lanes a row) go through LDS, a tile at a time in memory order (TileStream), 6.9 TB/s.  us a
//     call or solve, straight into registers / through LDS: 230M x 24 Hessian-vector 7110 / 6410; 5M x 18 136 and 128 (logistic and L2-SVM)
//     / 125 and 118, function/gradient 156 and 135 / 141 and 121, logistic solve 704 / 652; 10M x 9 137 / 126 and 161 / 151;
//   - rows over 16 lanes or more are loaded as they are, non-temporally: 240,000 x 512 181 / 160 us a Hessian-vector call, 200,003 x 257 82 / 75; but
//     60,000 x 512 (246 MB) 50 / 53, 40,000 x 127 22 / 24;
//   - rows of 1 to 8 columns, a lane a row, and of 33 to 64, eight lanes a row, are loaded ordinarily.  us a Hessian-vector call (logistic and L2-SVM),
//     ordinary / non-temporal loads: 20M x 2 98 and 68 / 113 and 110, 8M x 7 106 and 94 / 222 and 213, 8M x 8 115 and 103 / 163 and 159; 1.5M x 33 91 and 89
//     / 126 and 125, 1M x 57 102 and 101 / 142 and 142.  Not so even numbers from 40 on, whose 16-byte pieces make whole lines: 1.3M x 40 93 and
//     92 / 88 and 88, 1.2M x 48 101 and 100 / 91 and 91, 5M x 64 454 and 447 / 404 and 400; they are loaded like the others of eight lanes.
constexpr int64_t kOnceDoubles = 36'000'000;   // 288 MB
__host__ __device__ inline bool read_once(int64_t n, int64_t d) { return n * d > kOnceDoubles; }
constexpr bool tiles_stream(int L) { return L == 2 || L == 4; }

// A wave tile of RT = U * 64 / L rows.  A row is covered by L consecutive lanes; lane q of them holds the columns
// col(q, 0) .. col(q, E - 1): pieces of one or two columns (8 or 16 bytes) dealt to the L lanes in turn, so that one
// load instruction reads L consecutive pieces of a row and the next one the pieces behind them.  (With E consecutive columns
// per lane every instruction touches all cache lines of its rows and takes a part of each: a Hessian-vector pass over
// 200,003 x 257 took 82 us, this way 70 us; 3M x 25 173 us against 158 us a call.)  Step u covers the 64 / L consecutive
// rows u * RW + lane / L; steps of rows that lie U apart, which would make lane i the owner of row i, took 192 us
// against 162 us on 5M x 18.  The sum over a row's lanes is folded so that step u's total ends up in the lanes with
// lane % U == u (row_sum), which own the row: no exchange through LDS between the sums, the per-row work and the way back.
// (Tiles of matrices above 288 MB come through LDS by loads that write it directly, see TileStream: 118 to 125 us on 5M x 18.  Copied
// there through registers, a tile at a time and nothing under way meanwhile, they took 227 us.)
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

    // the same from the ballot of the owners, whose bits are in the order of the lanes: those of a row's U owners side by side
    __device__ static __forceinline__ uint64_t rows_of_ballot(uint64_t b)
    {
        static_assert(RT == kWave && U == L, "");
#pragma unroll
        for (int i = 1; i < U; i *= 2) {   // the even bits to the lower half, the odd ones to the upper half
            auto swap = [&](int by, uint64_t mask) { const uint64_t t = (b ^ (b >> by)) & mask; b ^= t ^ (t << by); };
            swap(1, 0x2222222222222222ull);
            swap(2, 0x0c0c0c0c0c0c0c0cull);
            swap(4, 0x00f000f000f000f0ull);
            swap(8, 0x0000ff000000ff00ull);
            swap(16, 0x00000000ffff0000ull);
        }
        return b;
    }

    // load the U x E block of this lane; out-of-range rows / columns read as zero.  rows: bit i clear = row row0 + i
    // is not needed (its coefficient is zero) and is not read at all
    __device__ static __forceinline__ void load(const double *__restrict__ X, int64_t n, int64_t d, int64_t row0,
                                                int lane, double (&x)[U][E], uint64_t rows = ~0ull)
    {
        if constexpr (L >= 16) {
            if (read_once(n, d)) {   // uniform
                load_as<true>(X, n, d, row0, lane, x, rows);
                return;
            }
        }
        load_as<false>(X, n, d, row0, lane, x, rows);
    }

    template <bool once>
    __device__ static __forceinline__ void load_as(const double *__restrict__ X, int64_t n, int64_t d, int64_t row0,
                                                   int lane, double (&x)[U][E], uint64_t rows)
    {
        const int q = lane % L, rl = lane / L;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t row = row0 + u * RW + rl;
            const bool rok = row < n && ((rows >> (u * RW + rl)) & 1u);
            const double *p = X + row * d;
            auto pg = (const __attribute__((address_space(1))) double *)p;
            if constexpr (once) asm volatile("" : "+v"(pg));   // (otherwise the compiler makes one ordinary load of this one and the other instance's)
            if (VEC) {
#pragma unroll
                for (int e = 0; e < E; e += 2) {
                    double2 t = make_double2(0.0, 0.0);
                    if constexpr (once) {
                        v2d o = v2d{0.0, 0.0};
                        if (rok && col(q, e) < d) o = __builtin_nontemporal_load((const __attribute__((address_space(1))) v2d *)(pg + col(q, e)));
                        t = make_double2(o.x, o.y);
                    } else if (rok && col(q, e) < d) t = *reinterpret_cast<const double2 *>(p + col(q, e));
                    x[u][e] = t.x;
                    x[u][e + 1] = t.y;
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) x[u][e] = !(rok && col(q, e) < d) ? 0.0 : once ? __builtin_nontemporal_load(pg + col(q, e)) : p[col(q, e)];
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
        if constexpr (U == 2) { c[0] = dpp_fetch<0xA0>(mine); c[1] = dpp_fetch<0xF5>(mine); }   // quad_perm [0,0,2,2], [1,1,3,3]
        if constexpr (U == 4) { c[0] = dpp_fetch<0x00>(mine); c[1] = dpp_fetch<0x55>(mine); c[2] = dpp_fetch<0xAA>(mine); c[3] = dpp_fetch<0xFF>(mine); }
    }

    // acc[e] summed over the lanes that hold the same columns, every one of which receives the sum: moves between lanes, no LDS (with
    // shuffles through LDS a solve over 20,000 x 24 took 49 us instead of 47)
    __device__ static __forceinline__ void sum_columns(double (&acc)[E])
    {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if constexpr (L <= 1) acc[e] += dpp_fetch<0xB1>(acc[e]);
            if constexpr (L <= 2) acc[e] += dpp_fetch<0x4E>(acc[e]);
            if constexpr (L <= 4) acc[e] += other_quad_of_8(acc[e]);
            if constexpr (L <= 8) acc[e] += dpp_fetch<0x128>(acc[e]);
            if constexpr (L <= 16) acc[e] = add_row_pairs(acc[e]);
            if constexpr (L <= 32) acc[e] = add_halves(acc[e]);
        }
    }

    // ... then over the workgroup's wavefronts (`waves` of them): column c goes to out[c * stride].  lds: waves * E * L doubles that
    // nothing else uses any more.
    __device__ static __forceinline__ void flush(double (&acc)[E], int64_t d, int lane, int wv, int waves, double *lds,
                                                 double *__restrict__ out, int64_t stride)
    {
        sum_columns(acc);
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

// Tiles of 64 rows through LDS: ask() has the wavefront's next tile copied there by loads that write LDS directly, a kilobyte in memory
// order each, and take() reads it into the registers of Tile.  A tile of which a part is past the end, or that was not asked for, is
// loaded as ever.  One buffer a wavefront: it is asked for again as soon as it has been read, so that eight wavefronts a CU
// have 512 d bytes each on their way all the time, during the arithmetic as well.
template <int E, int L, int U, bool VEC>
struct TileStream {
    using T = Tile<E, L, U, VEC>;
    double *buf;          // the wavefront's 64 d doubles, 16-byte aligned; null: every tile is loaded straight into registers
    bool there = false;   // the tile asked for is in LDS or on its way

    static constexpr int64_t bytes(int64_t d, int waves) { return 512 * d * waves; }
    __device__ __forceinline__ TileStream(double *lds, int64_t d)   // lds: the workgroup's, or null
        : buf(lds ? lds + 64 * d * __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : nullptr) {}

    // nothing may be on its way but what take() has waited for
    __device__ __forceinline__ void ask(const double *__restrict__ X, int64_t n, int64_t d, int64_t tile, bool wanted)
    {
        if constexpr (tiles_stream(L)) {
            static_assert(T::RT == kWave, "");
            there = __builtin_amdgcn_readfirstlane((int)(buf != nullptr && wanted && (tile + 1) * kWave <= n));
            if (!there) return;
            const int lane = threadIdx.x & (kWave - 1);
            const double *src = X + tile * kWave * d + 2 * lane;
            const int whole = (int)(d / 2);   // kilobytes
#pragma unroll
            for (int k = 0; k < (E * L + 1) / 2; ++k)
                if (k < whole) copy(src + 128 * k, buf + 128 * k);
            if ((d & 1) && lane < kWave / 2) copy(src + 128 * whole, buf + 128 * whole);
        }
    }

    __device__ __forceinline__ void take(const double *__restrict__ X, int64_t n, int64_t d, int64_t tile, int lane, double (&x)[U][E], uint64_t rows = ~0ull)
    {
        if (!tiles_stream(L) || !there) {
            T::load(X, n, d, tile * T::RT, lane, x, rows);
            wait_loads();   // here, or the compiler waits for these registers where both ways have joined, behind the next ask()
            return;
        }
        wait_loads();
        const int q = lane % L, rl = lane / L;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double *p = buf + (u * T::RW + rl) * d;
            if (VEC) {
#pragma unroll
                for (int e = 0; e < E; e += 2) {
                    v2d t = v2d{0.0, 0.0};
                    if (T::col(q, e) < d) t = *reinterpret_cast<const v2d *>(p + T::col(q, e));
                    x[u][e] = t.x;
                    x[u][e + 1] = t.y;
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) x[u][e] = T::col(q, e) < d ? p[T::col(q, e)] : 0.0;
            }
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): in registers, before the buffer is asked for again
        asm volatile("" ::: "memory");
        there = false;
        if (rows != ~0ull) {   // uniform; rows that are not needed count as zeros, whatever lies in them
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool needed = (rows >> (u * T::RW + rl)) & 1u;
#pragma unroll
                for (int e = 0; e < E; ++e) x[u][e] = needed ? x[u][e] : 0.0;
            }
        }
    }

    __device__ static __forceinline__ void wait_loads()
    {
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        asm volatile("" ::: "memory");
    }

private:
    __device__ static __forceinline__ void copy(const double *from, double *to)
    {
        constexpr int kNonTemporal = 2;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from, (__attribute__((address_space(3))) void *)to, 16, 0, kNonTemporal);
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
