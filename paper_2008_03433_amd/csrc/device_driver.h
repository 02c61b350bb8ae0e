// Algorithm 1 of the paper on the device: the state of problems that advance without the host, and the step a problem
// takes when the product it was waiting for is there.  Used by the multi-problem pass (batch.hip) and by solves of one dense
// problem (k_dense_solve).  The vectors have d <= 32 entries, one lane each.
#pragma once

#include "device_util.h"

namespace tron {

constexpr int kBatchMax = TRON_BATCH_MAX;
constexpr int kVecPad = TRON_BATCH_MAX_D;   // doubles per stored vector
static_assert(kVecPad <= kWave, "one lane per vector entry");

enum { MODE_IDLE = 0, MODE_HV = 1, MODE_FG = 2, MODE_DIAG = 3 };   // MODE_DIAG: column sums of D_i x_ij^2 (the Hessian diagonal)
enum { PH_DONE = 0, PH_ONESHOT, PH_REF, PH_START, PH_CG, PH_TRIAL, PH_DIAG0, PH_DIAG };
enum { BEGIN_SOLVE = 0, BEGIN_FG, BEGIN_HV };

// request of the next pass: written by the begin / advance kernels, read by the pass
struct BatchCtl {
    int32_t mode[kBatchMax];    // MODE_*
    int32_t dslot[kBatchMax];   // which of the problem's two D buffers the pass reads (MODE_HV) or writes (MODE_FG)
    double vec[kBatchMax][kVecPad];   // v (MODE_HV) or w (MODE_FG), zero past d
};

struct ProbScalars {
    int32_t phase, status, converged, outer, cg_total, n_fun, n_grad, n_hv, cg_it, onb, dcur, trace_len;
    double C, f, gnorm, gnorm0, delta, rr, pred, snorm, out_scal;
    double gscaled;   // what the inner solver measures its residual against: |g|, or sqrt(g.M^-1 g) with a preconditioner
};

// solver state of one problem (device memory)
struct ProbState {
    ProbScalars sc;
    double w[kVecPad], wnew[kVecPad], g[kVecPad], s[kVecPad], r[kVecPad], p[kVecPad];
    double M[kVecPad];   // diagonal preconditioner (1 - a) I + a diag(H) of the current iterate (used when blend > 0)
};

struct SolveParams {
    int loss, max_outer, max_cg, trace_cap;
    double eps, xi;
    double *out;    // device, K x d: the final iterates of a solve, or the products of a single call (may be null)
    double blend;   // 0: plain CG; a in (0, 1]: CG preconditioned by M = (1 - a) I + a diag(H), rebuilt at every accepted iterate
};

struct BatchC { double v[kBatchMax]; };

// What the host reads while the rounds run (pinned host memory, written by the kernels): per problem the number of the last
// round it has seen times four plus the mode of its next request, and, once it is idle, its results.
struct BatchHost {
    int64_t stamp[kBatchMax];
    int64_t finished;   // a solve in one launch has its results
    ProbScalars sc[kBatchMax];
};

// Device memory and pinned host memory of K problems driven from the device
struct DriverState {
    BatchCtl *ctl = nullptr;
    ProbState *st = nullptr;
    BatchHost *host = nullptr, *host_dev = nullptr;         // pinned; its device address
    tron_trace_rec *trace = nullptr, *trace_dev = nullptr;  // pinned, K x trace_cap
    int trace_cap = 0;
    int64_t rounds = 0;   // enqueued so far
    int create(int K, hipStream_t st);
    int ensure_trace(int K, int cap);
    void release();
};

// ------------------------------------------------------------------ per-problem steps on the device
// Every lane of the wavefront executes every statement (the sums run over all 64 lanes); lanes at or past d hold zeros
// and their memory accesses are masked by `in`.
__device__ __forceinline__ double dot64(double a, double b) { return wave_sum(a * b); }

struct Request {
    int mode, slot;
    double vec;   // this lane's entry of the vector
};

// Start of the truncated CG iteration at the current iterate: s = 0, r = -g, p = r (preconditioned: p = r / M, and the
// residual is measured by r.M^-1 r); the first product is H p.  m: this lane's entry of M, 1 without a preconditioner.
__device__ __forceinline__ Request cg_begin(ProbState &S, ProbScalars &sc, int j, bool in, double g, double m)
{
    const double p0 = -g / m;
    if (in) {
        S.s[j] = 0.0;
        S.r[j] = -g;
        S.p[j] = p0;
    }
    sc.rr = sc.gscaled * sc.gscaled;
    sc.cg_it = 0;
    sc.onb = 0;
    sc.phase = PH_CG;
    return Request{MODE_HV, sc.dcur, p0};
}

// End of the inner iteration: trial point w + s and the model's reduction pred = -q(s) = -1/2 (g.s - s.r);
// the next pass evaluates f and the gradient there, D going to the problem's other buffer.
__device__ __forceinline__ Request cg_end(ProbState &S, ProbScalars &sc, int j, bool in, double s, double r, double m)
{
    const double w = in ? S.w[j] : 0.0, g = in ? S.g[j] : 0.0;
    const double wnew = w + s;
    const double gs = dot64(g, s), sr = dot64(s, r);
    sc.snorm = sqrt(dot64(m * s, s));   // the length the radius rules use: the M-norm of the iteration
    sc.pred = -0.5 * (gs - sr);
    if (in) S.wnew[j] = wnew;
    sc.phase = PH_TRIAL;
    return Request{MODE_FG, 1 - sc.dcur, wnew};
}

__device__ __forceinline__ void finish(ProbScalars &sc, int status)
{
    sc.status = status;
    sc.converged = (status == TRON_OK) ? 1 : 0;
    sc.phase = PH_DONE;
}

// Problem k's step, by one wavefront.  mode = the request the pass just served, cj its column sum of this lane's column,
// loss_sum the loss sum; stamp = the number of the round.  host, trace, P.out null: nothing is reported there.  The rules are those of the single-problem driver (Algorithm 1
// with Steihaug's truncated CG), lane j holding entry j of every vector.
__device__ __forceinline__ void advance_problem(const int k, const int mode, const int64_t d, const double cj, const double loss_sum, BatchCtl *ctl, ProbState *st,
                                                const SolveParams &P, tron_trace_rec *trace, BatchHost *host, const int64_t stamp)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (mode == MODE_IDLE) {
        if (lane == 0) __hip_atomic_store(&host->stamp[k], (stamp << 2) | MODE_IDLE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    ProbState &S = st[k];
    ProbScalars sc = S.sc;   // every lane works on a copy; lane 0 writes it back
    const bool in = lane < d;
    const int j = in ? lane : 0;
    const double C = sc.C;
    const bool one_shot = sc.phase == PH_ONESHOT;
    const double u = in ? ctl->vec[k][j] : 0.0;     // entry j of the vector the pass used
    const double o = in ? fma(C, cj, u) : 0.0;   // entry j of  v + C X^T(D(Xv))  or of  w + C X^T zhat
    Request next{MODE_IDLE, sc.dcur, 0.0};
    const double eta0 = 1e-4, eta1 = 0.25, eta2 = 0.75, sig2 = 0.5, sig3 = 4.0;
    const bool precond = P.blend > 0.0;
    // this lane's entry of the preconditioner; 1 without one (and past d), which leaves every product below unchanged
    double m = (precond && in && sc.phase != PH_ONESHOT) ? S.M[j] : 1.0;

    if (mode == MODE_DIAG) {
        // cj = sum_i D_i x_ij^2 at the current iterate: M = (1 - a) + a (1 + C cs) = 1 + a C cj, then the inner solve starts
        m = in ? fma(P.blend * C, cj, 1.0) : 1.0;
        if (in) S.M[j] = m;
        const double g = in ? S.g[j] : 0.0;
        sc.gscaled = sqrt(dot64(g, g / m));
        if (sc.phase == PH_DIAG0) sc.delta = sc.gscaled;   // Delta_0 = sqrt(g.M^-1 g)
        next = cg_begin(S, sc, j, in, g, m);
    } else if (mode == MODE_HV) {
        const double pHp = dot64(u, o);
        if (sc.phase == PH_ONESHOT) {
            sc.out_scal = pHp;
            sc.phase = PH_DONE;
        } else {   // PH_CG: u is the direction p
            double s = in ? S.s[j] : 0.0, r = in ? S.r[j] : 0.0;
            sc.cg_it += 1;
            sc.n_hv += 1;
            sc.cg_total += 1;
            const double alpha = sc.rr / pHp;
            const double pp = dot64(m * u, u), sp = dot64(m * s, u), ss = dot64(m * s, s);
            bool end = false;
            if (sqrt(ss + alpha * (2.0 * sp + alpha * pp)) >= sc.delta) {
                // to the boundary along p
                const double gap = sc.delta * sc.delta - ss;
                const double rad = sqrt(sp * sp + pp * gap);
                const double tau = (sp >= 0.0) ? gap / (sp + rad) : (rad - sp) / pp;
                s = fma(tau, u, s);
                r = fma(-tau, o, r);
                sc.onb = 1;
                end = true;
            } else {
                s = fma(alpha, u, s);
                r = fma(-alpha, o, r);
                const double zr = r / m;
                const double rr_new = dot64(r, zr);
                const double beta = rr_new / sc.rr;
                sc.rr = rr_new;
                if (sqrt(rr_new) <= P.xi * sc.gscaled || sc.cg_it >= P.max_cg) {
                    end = true;
                } else {
                    const double p = fma(beta, u, zr);
                    if (in) S.p[j] = p;
                    next = Request{MODE_HV, sc.dcur, p};
                }
            }
            if (in) {
                S.s[j] = s;
                S.r[j] = r;
            }
            if (end) next = cg_end(S, sc, j, in, s, r, m);
        }
    } else {   // MODE_FG: u is the point, o the gradient there
        const double f = 0.5 * dot64(u, u) + C * loss_sum;
        const double gn = sqrt(dot64(o, o));
        if (sc.phase == PH_ONESHOT) {
            sc.out_scal = f;
            sc.phase = PH_DONE;
        } else if (sc.phase == PH_REF) {
            // the gradient at w = 0 is the reference of the stopping test; now the starting point itself
            sc.gnorm0 = gn;
            sc.n_fun += 1;
            sc.n_grad += 1;
            sc.phase = PH_START;
            next = Request{MODE_FG, sc.dcur, in ? S.w[j] : 0.0};
        } else if (sc.phase == PH_START) {
            sc.f = f;
            sc.gnorm = gn;
            if (in) S.g[j] = o;
            sc.n_fun += 1;
            sc.n_grad += 1;
            if (sc.gnorm0 == 0.0) sc.gnorm0 = gn;
            sc.delta = gn;
            sc.gscaled = gn;
            if (gn <= P.eps * sc.gnorm0) finish(sc, TRON_OK);
            else if (precond) {   // the Hessian diagonal at this iterate first
                sc.phase = PH_DIAG0;
                next = Request{MODE_DIAG, sc.dcur, 0.0};
            } else next = cg_begin(S, sc, j, in, o, 1.0);
        } else {   // PH_TRIAL
            sc.n_fun += 1;
            const double ared = sc.f - f;
            const bool noise = fabs(ared) <= 1e-12 * fabs(sc.f) && sc.pred <= 1e-12 * fabs(sc.f);
            const double sigma = noise ? 1.0 : ared / sc.pred;
            const double gnorm_before = sc.gnorm;
            if (sigma < eta1) sc.delta = sig2 * fmin(sc.snorm, sc.delta);
            else if (sigma < eta2) { /* unchanged */ }
            else sc.delta = fmin(sig3 * sc.delta, fmax(sc.delta, sig3 * sc.snorm));
            const bool accepted = sigma > eta0;
            double g = in ? S.g[j] : 0.0;
            if (accepted) {
                if (in) {
                    S.w[j] = u;
                    S.g[j] = o;
                }
                g = o;
                sc.dcur = 1 - sc.dcur;   // the Hessian now uses D at the accepted point
                sc.f = f;
                sc.gnorm = gn;
                sc.gscaled = gn;
                sc.n_grad += 1;
            }
            sc.outer += 1;
            if (trace && sc.trace_len < P.trace_cap) {
                if (lane == 0) {
                    tron_trace_rec &t = trace[(int64_t)k * P.trace_cap + sc.trace_len];
                    t.iter = sc.outer; t.cg_iters = sc.cg_it; t.accepted = accepted ? 1 : 0; t.on_boundary = sc.onb;
                    t.f = sc.f; t.gnorm = sc.gnorm; t.delta = sc.delta; t.ared = ared; t.pred = sc.pred; t.snorm = sc.snorm;
                }
                sc.trace_len += 1;
            }
            if (accepted && sc.gnorm <= P.eps * sc.gnorm0) finish(sc, TRON_OK);
            else if (sc.pred <= 0.0 || (noise && sc.gnorm >= gnorm_before)) finish(sc, TRON_EMAXITER);
            else if (sc.outer >= P.max_outer) finish(sc, TRON_EMAXITER);
            else if (precond && accepted) {   // the iterate moved: its Hessian diagonal, then the inner solve
                sc.phase = PH_DIAG;
                next = Request{MODE_DIAG, sc.dcur, 0.0};
            } else next = cg_begin(S, sc, j, in, g, m);   // after a rejected step M and sqrt(g.M^-1 g) still hold
        }
    }
    if (lane < kVecPad) ctl->vec[k][lane] = in ? next.vec : 0.0;
    if (lane == 0) {
        ctl->mode[k] = next.mode;
        ctl->dslot[k] = next.slot;
        S.sc = sc;
        if (host && sc.phase == PH_DONE) host->sc[k] = sc;
    }
    if (sc.phase == PH_DONE && in && P.out) store_shared(P.out + (int64_t)k * d + j, one_shot ? o : S.w[j]);
    // running or not, for the host that enqueues rounds meanwhile (see drive_rounds); of a problem that is done, after its results
    if (sc.phase == PH_DONE) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (host && lane == 0) __hip_atomic_store(&host->stamp[k], (stamp << 2) | next.mode, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    } else if (host && lane == 0) {
        __hip_atomic_store(&host->stamp[k], (stamp << 2) | next.mode, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// First request of problem k, by one wavefront.  what = BEGIN_SOLVE: state reset, w0 = IN[k]; when w0 is not zero the gradient
// at zero is evaluated first (it is the reference of the stopping test).  BEGIN_FG / BEGIN_HV: a single product with IN[k],
// using the problem's current D buffer.
__device__ __forceinline__ void begin_problem(const int k, const int what, const int64_t d, const double *__restrict__ IN, const double C,
                                              BatchCtl *ctl, ProbState *st)
{
    const int lane = threadIdx.x & (kWave - 1);
    ProbState &S = st[k];
    const bool in = lane < d;
    const double x = in ? IN[(int64_t)k * d + lane] : 0.0;
    ProbScalars sc = S.sc;
    sc.C = C;
    Request next{MODE_IDLE, 0, 0.0};
    if (what == BEGIN_SOLVE) {
        sc.status = TRON_EMAXITER;
        sc.converged = sc.outer = sc.cg_total = sc.n_fun = sc.n_grad = sc.n_hv = sc.cg_it = sc.onb = sc.trace_len = 0;
        sc.dcur = 0;
        sc.f = sc.gnorm = sc.gnorm0 = sc.delta = sc.rr = sc.pred = sc.snorm = sc.out_scal = sc.gscaled = 0.0;
        if (in) S.w[lane] = x;
        const bool nonzero = __ballot(x != 0.0) != 0;
        sc.phase = nonzero ? PH_REF : PH_START;
        next = Request{MODE_FG, 0, nonzero ? 0.0 : x};
    } else {
        sc.phase = PH_ONESHOT;
        next = Request{what == BEGIN_FG ? MODE_FG : MODE_HV, sc.dcur, x};
    }
    if (lane < kVecPad) ctl->vec[k][lane] = in ? next.vec : 0.0;
    if (lane == 0) {
        ctl->mode[k] = next.mode;
        ctl->dslot[k] = next.slot;
        S.sc = sc;
    }
}

}  // namespace tron
