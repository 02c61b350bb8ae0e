// Device-side helpers: wavefront / workgroup sums and the per-instance loss terms.
#pragma once

#include "common.h"

namespace tron {

// Cross-lane moves through the DPP data path (a few cycles) instead of ds_bpermute (an LDS round trip):
//   0xB1 = quad_perm [1,0,3,2] (lane ^ 1), 0x4E = quad_perm [2,3,0,1] (lane ^ 2),
//   0x141 = row_half_mirror (lane i <-> 7-i inside each group of 8), 0x140 = row_mirror (i <-> 15-i inside 16).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    hi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// The same where every lane takes part: nothing has to lie in the result's registers before, which dpp_move copies v to
template <int CTRL>
__device__ __forceinline__ double dpp_fetch(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double read_lane(double v, int lane)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// A zero that the compiler takes for lane-dependent: an address formed with it is read with a vector load.  A scalar load
// would be counted by the same counter as the LDS operations, so the next wait for LDS would also wait for memory.
__device__ __forceinline__ int lane_zero()
{
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    return zero;
}

// Two values to add over pairs of lanes, of which each lane of a pair keeps one: lanes with `odd` clear return a summed over
// the pair, the others b.  CTRL moves each lane's partner to it (0xB1: lane ^ 1, 0x4E: lane ^ 2).
template <int CTRL>
__device__ __forceinline__ double fold(double a, double b, int odd)
{
    const double keep = odd ? b : a, give = odd ? a : b;
    return keep + dpp_move<CTRL>(give);
}

// v of lane ^ 4: row_shr:4 into the upper quad of every eight lanes, row_shl:4 into the lower one
__device__ __forceinline__ double other_quad_of_8(double v)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    int a = __builtin_amdgcn_update_dpp(lo, lo, 0x114, 0xf, 0xa, false);
    a = __builtin_amdgcn_update_dpp(a, lo, 0x104, 0xf, 0x5, false);
    int b = __builtin_amdgcn_update_dpp(hi, hi, 0x114, 0xf, 0xa, false);
    b = __builtin_amdgcn_update_dpp(b, hi, 0x104, 0xf, 0x5, false);
    return __hiloint2double(b, a);
}

// v + (v of lane ^ 16), v + (v of lane ^ 32): permlane16_swap / permlane32_swap of a value with itself give both operands
__device__ __forceinline__ double add_row_pairs(double v)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double add_halves(double v)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}

// Sum over aligned groups of 2 / 4 / 8 / 16 consecutive lanes; every lane of a group receives its total.
__device__ __forceinline__ double sum2(double v) { return v + dpp_move<0xB1>(v); }
__device__ __forceinline__ double sum4(double v) { v = sum2(v); return v + dpp_move<0x4E>(v); }
__device__ __forceinline__ double sum8(double v) { v = sum4(v); return v + dpp_move<0x141>(v); }
__device__ __forceinline__ double sum16(double v) { v = sum8(v); return v + dpp_move<0x140>(v); }

// Sum over the 64 lanes of a wavefront; every lane receives the total.  Fixed order.
__device__ __forceinline__ double wave_sum(double v)
{
    v = sum16(v);
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Sum over aligned groups of `g` consecutive lanes (g a power of two <= 64); every lane of a group gets its total.
__device__ __forceinline__ double group_sum(double v, int g)
{
    if (g == 1) return v;
    if (g == 2) return sum2(v);
    if (g == 4) return sum4(v);
    if (g == 8) return sum8(v);
    v = sum16(v);
    if (g == 16) return v;
    if (g == 32) return v + __shfl_xor(v, 16, kWave);
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// *a += v with the LDS add instruction: one operation instead of a read, an add and a write, and nothing to wait for.
// Used where no two lanes address the same word between two barriers and a lane's own additions to one word are issued
// in program order (LDS operations of a wavefront complete in order), so the sum is built in a fixed order.
__device__ __forceinline__ void lds_add(double *a, double v)
{
    (void)__hip_atomic_fetch_add(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---- inclusive scans over the 64 lanes of a wavefront, through DPP (no LDS).
// Steps: row_shr 1, 2, 4, 8 inside each row of 16 lanes, then row_bcast:15 into rows 1 and 3 (lane 15 of the row
// before), then row_bcast:31 into rows 2 and 3.  A lane that has no source in a step keeps the identity it passes in.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_int(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}

// c := c[0] + ... + c[lane]
__device__ __forceinline__ int wave_scan_add(int c)
{
    c += dpp_int<0x111, 0xf>(c);
    c += dpp_int<0x112, 0xf>(c);
    c += dpp_int<0x114, 0xf>(c);
    c += dpp_int<0x118, 0xf>(c);
    c += dpp_int<0x142, 0xa>(c);
    c += dpp_int<0x143, 0xc>(c);
    return c;
}

// Segmented sum: every lane holds (t, h) = (sum of the open run at its end, whether a run ended inside it).
// Afterwards t = t[lane] + the t of the lanes before it back to, and including, the nearest one with h set, and
// h = whether any lane up to this one had h set.  The operator (ta,ha)+(tb,hb) = (hb ? tb : ta+tb, ha|hb) is
// associative, so the tree order above applies.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void seg_scan_step(double &t, int &h)
{
    // h is 0 or 1: the mask keeps the incoming sum only while no run has ended up to this lane (t + 0.0 is t)
    const int open = h - 1;
    const int lo = dpp_int<CTRL, ROW_MASK>(__double2loint(t)) & open;
    const int hi = dpp_int<CTRL, ROW_MASK>(__double2hiint(t)) & open;
    const int sh = dpp_int<CTRL, ROW_MASK>(h);
    t += __hiloint2double(hi, lo);
    h |= sh;
}

__device__ __forceinline__ void wave_seg_scan(double &t, int &h)
{
    seg_scan_step<0x111, 0xf>(t, h);
    seg_scan_step<0x112, 0xf>(t, h);
    seg_scan_step<0x114, 0xf>(t, h);
    seg_scan_step<0x118, 0xf>(t, h);
    seg_scan_step<0x142, 0xa>(t, h);
    seg_scan_step<0x143, 0xc>(t, h);
}

// value of the lane before (lane 0 receives 0): wave_shr:1
__device__ __forceinline__ double lane_before(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ int lane_before(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, false); }

// Sum over the workgroup (kBlock threads); valid in thread 0.  `lds` holds kWavesPerBlock doubles
// and may be reused right after the call returns (the trailing barrier orders it).
__device__ __forceinline__ double block_sum(double v, double *lds)
{
    v = wave_sum(v);
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    if (lane == 0) lds[wv] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) t += lds[k];
    }
    __syncthreads();
    return t;
}

// ---- sums that one workgroup leaves for the workgroup that finishes last
// They are written through to where every XCD sees them (a relaxed store of device scope), and the wavefront that wrote
// them waits for the stores before it draws the ticket; the reader uses loads of device scope.  A fence of device scope
// (__threadfence) would do as well, but it writes back the XCD's whole L2 for every workgroup: a pass over 1M x 24 rows by 512
// workgroups took 59 us that way, by 2048 workgroups 119 us.
// Solves of sparse problems in one launch (csr_solve.hip) read what was stored this way with ordinary loads.  They rely on the L2 taking a
// store to a line that it does not hold without fetching the line's other bytes (a mask says which bytes it has): the next read
// fetches the line, after all have written.  The memory model does not promise it; were it otherwise, a solve in one launch and the same one with a
// launch per step, whose caches start empty, would differ, and the tests hold their bits together.
template <typename T>
__device__ __forceinline__ void store_shared(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double load_shared(const double *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// this wavefront's stores have arrived where they go to
__device__ __forceinline__ void stores_arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// For the host: a scalar, and the flag behind what this wavefront has stored (called by all of it; its lane 0 writes)
__device__ __forceinline__ void store_host(double *p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
__device__ __forceinline__ void post_flag(const HostFlag &f)
{
    if (!f.word) return;
    stores_arrived();
    if ((threadIdx.x & (kWave - 1)) == 0) __hip_atomic_store(f.word, f.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// True in every thread of the workgroup that draws the last of the launch's tickets.  Called by all threads; the workgroup's
// sums were stored by wavefront 0.  The counter is the only thing touched by a read-modify-write; the caller clears it.
__device__ __forceinline__ bool last_workgroup(unsigned *ticket)
{
    __shared__ int is_last;
    if (threadIdx.x < kWave) {
        stores_arrived();
        if (threadIdx.x == 0) is_last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    }
    __syncthreads();
    return is_last;
}

// Second reduction stage inside the producing kernel (see Finish in common.h).  Every thread of every workgroup calls it
// after thread 0 has stored the workgroup's partial sums (NSLOTS of them, `stride` apart; store_shared).  The workgroup that
// draws the last ticket adds the partial sums of all workgroups (and `extra` more behind them) -- in the order and with the
// arithmetic of k_reduce_final, so the result does not depend on which workgroup that is -- writes the scalars and clears the
// counter for the next kernel on the stream.
template <int NSLOTS>
__device__ __forceinline__ void finish_partials(const Finish &f, const double *partials, int stride, double *lds, int extra = 0)
{
    if (!f.ticket || !last_workgroup(f.ticket)) return;
    const int count = (int)gridDim.x + extra;
#pragma unroll
    for (int s = 0; s < NSLOTS; ++s) {
        const double *p = partials + (int64_t)s * stride;
        double acc = 0.0;
        for (int b = threadIdx.x; b < count; b += kBlock) acc += load_shared(p + b);
        acc = block_sum(acc, lds);
        if (threadIdx.x == 0) {
            f.scal[f.first + s] = acc;
            f.scal_copy[f.first + s] = acc;
        }
    }
    if (threadIdx.x == 0) *f.ticket = 0u;
}

// log(1 + e) for 0 <= e <= 1, as 2 atanh(u) with u = e / (2 + e) <= 1/3: the odd series in u up to u^31 (the first
// term left out is below 2e-17 of the sum).  Within 2 ulp of the exact value (4.2e-16 relative at worst over 2.6M
// arguments e = exp(-t), t in [0, 600], against extended precision on the host; the library's general-argument routine:
// 1.2e-16) at about a third of that routine's instructions.  For kernels whose lanes see few rows; the others use LossSum.
__device__ __forceinline__ double log1p_unit(double e)
{
    const double u = e / (2.0 + e), w = u * u;
    double p = 1.0 / 31.0;
    p = fma(p, w, 1.0 / 29.0);
    p = fma(p, w, 1.0 / 27.0);
    p = fma(p, w, 1.0 / 25.0);
    p = fma(p, w, 1.0 / 23.0);
    p = fma(p, w, 1.0 / 21.0);
    p = fma(p, w, 1.0 / 19.0);
    p = fma(p, w, 1.0 / 17.0);
    p = fma(p, w, 1.0 / 15.0);
    p = fma(p, w, 1.0 / 13.0);
    p = fma(p, w, 1.0 / 11.0);
    p = fma(p, w, 1.0 / 9.0);
    p = fma(p, w, 1.0 / 7.0);
    p = fma(p, w, 1.0 / 5.0);
    p = fma(p, w, 1.0 / 3.0);
    p = fma(p, w, 1.0);
    return 2.0 * u * p;
}

// e^x for x <= 0 (NaN stays NaN): x = k ln 2 + r with |r| <= ln 2 / 2, ln 2 in two parts, and e^r = 1 + r + r^2 q(r) with q the
// interpolation polynomial in the eleven Chebyshev nodes of that interval (error of the whole 3.4e-19 relative).  At worst 1.5e-16
// relative to extended precision over 3M arguments in [-700, 0].  A general routine's tests for overflow are left out.
__device__ __forceinline__ double exp_nonpositive(double x)
{
    const double c = x < -750.0 ? -750.0 : x;   // e^-750 is 0 in fp64 already
    const double k = __builtin_rint(c * 1.4426950408889634);
    const double r = fma(k, -2.3190468138462996e-17, fma(k, -0.6931471805599453, c));
    double q = 2.0914686968086876e-09;
    q = fma(q, r, 2.5105217004720745e-08);
    q = fma(q, r, 2.75572736431103e-07);
    q = fma(q, r, 2.7557255400206422e-06);
    q = fma(q, r, 2.4801587325547743e-05);
    q = fma(q, r, 0.00019841269874820627);
    q = fma(q, r, 0.0013888888888883748);
    q = fma(q, r, 0.008333333333326136);
    q = fma(q, r, 0.04166666666666667);
    q = fma(q, r, 0.1666666666666667);
    q = fma(q, r, 0.5);
    return ldexp(1.0 + fma(r * r, q, r), (int)k);
}

// 1 / x for x in [1, 2]: two Newton steps from the hardware's approximation (24 bits at least).  The second one corrects a value that is within
// an ulp or two by a residual known to 2^-52 of itself, so what is rounded is the quotient to 2^-50 of an ulp: the division's result but
// for quotients that close to the middle between two numbers.  No scaling and no special cases: a division is eleven instructions.
__device__ __forceinline__ double reciprocal_1_2(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// What a row adds to the sum of the losses (LossSum): alpha = lin + log(1 + e), e = 0 for the L2-SVM.
struct LossTerm {
    double lin, e;
};

// Per-instance terms at margin z with label y (Table 1 and Appendix E of the paper):
//   logistic:  t = y z, h = 1/(1+exp(-t));  alpha = log(1+exp(-t)),  zhat = (h-1) y,  D = h (1-h)
//   L2-SVM:    m = 1 - y z;  active iff m > 0;  alpha = max(0,m)^2,  zhat = 2 (z-y) [active],  D = 2 [active]
// The exponential is only taken of a non-positive argument, and 1-h is formed without cancellation.
template <int LOSS>
__device__ __forceinline__ void loss_terms_dev(double z, double y, LossTerm &a, double &zhat, double &D)
{
    if (LOSS == TRON_LOSS_LR) {
        const double t = y * z;
        const double e = exp_nonpositive(-fabs(t));
        const double inv = reciprocal_1_2(1.0 + e);
        const double big = inv, small = e * inv;   // h and 1-h in some order
        a.e = e;
        a.lin = (t >= 0.0) ? 0.0 : -t;
        zhat = -((t >= 0.0) ? small : big) * y;
        D = big * small;
    } else {
        const double m = 1.0 - y * z;
        const bool act = m > 0.0;
        a.e = 0.0;
        a.lin = act ? m * m : 0.0;
        zhat = act ? 2.0 * (z - y) : 0.0;
        D = act ? 2.0 : 0.0;
    }
}

// the same with the row's loss formed at once
template <int LOSS>
__device__ __forceinline__ void loss_terms_dev(double z, double y, double &alpha, double &zhat, double &D)
{
    LossTerm a;
    loss_terms_dev<LOSS>(z, y, a, zhat, D);
    alpha = LOSS == TRON_LOSS_LR ? log1p_unit(a.e) + a.lin : a.lin;
}

// The sum of a lane's losses.  The logarithms of the logistic loss are taken of their product, once: the sum of log(1 + e_i) is
// log(1 + p) with 1 + p = prod (1 + e_i), and p -> p + e + p e adds positive numbers only, so small e lose nothing.  (One series a
// row, thirty instructions of 85, was the largest part of the logistic terms: a function/gradient call of twelve problems over
// 20M x 24 rows takes 1.75 ms instead of 2.1.)
template <int LOSS>
struct LossSum {
    double lin = 0.0, p = 0.0;
    __device__ __forceinline__ void add(const LossTerm &a)
    {
        lin += a.lin;
        if constexpr (LOSS == TRON_LOSS_LR) p = fma(p, a.e, p + a.e);
    }
    // to be called after at most kAdds additions: keeps p below 2^512
    static constexpr int kAdds = 256;
    __device__ __forceinline__ void scale()
    {
        if constexpr (LOSS == TRON_LOSS_LR) {
            const bool large = p > 0x1p256;
            p = large ? fma(p, 0x1p-256, -1.0) : p;
            lin += large ? 256.0 * 0.6931471805599453 : 0.0;
        }
    }
    __device__ __forceinline__ double value() const { return LOSS == TRON_LOSS_LR ? lin + log1p(p) : lin; }
};

}  // namespace tron
