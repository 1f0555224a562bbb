// dl_krylov.hpp -- the per-right-hand-side scalar steps of BiCGStab, shared by
// the batched solver's scalar kernels and the one-kernel solver of small
// lattices.  Each takes sums over the right-hand side's sites.
#pragma once

#include "dl_internal.hpp"

namespace dl {

__device__ __forceinline__ void cdiv(const double a[2], const double b[2], double out[2])
{
    double d = b[0] * b[0] + b[1] * b[1];
    double re = (a[0] * b[0] + a[1] * b[1]) / d, im = (a[1] * b[0] - a[0] * b[1]) / d;
    out[0] = re;
    out[1] = im;
}
__device__ __forceinline__ void cmul(const double a[2], const double b[2], double out[2])
{
    double re = a[0] * b[0] - a[1] * b[1], im = a[0] * b[1] + a[1] * b[0];
    out[0] = re;
    out[1] = im;
}

// (Re)start of the recursion: rho = (rhat, r) (with rhat = r, so |r|^2 is its
// real part), alpha = omega = 1.
__device__ __forceinline__ void bicg_rho_step(KState &s, const double rn[2])
{
    s.rho[0] = rn[0];
    s.rho[1] = rn[1];
    s.alpha[0] = s.omega[0] = 1.0;
    s.alpha[1] = s.omega[1] = 0.0;
    s.beta[0] = s.beta[1] = 0.0;
    s.rr = rn[0];
    s.maxrr = rn[0];
    if (!isfinite(rn[0]) || !isfinite(rn[1])) s.nonfinite = 1;
}

// omega = (t, s) / |t|^2 from d = (t, s), |t|^2, (rhat, t), (rhat, s); the next
// rho by linearity of r = s - omega t, rho' = (rhat, s) - omega (rhat, t);
// beta = (rho' / rho) (alpha / omega).  Each dot is taken directly from the
// vectors of this iteration: nothing accumulates across iterations.  (rhat, s)
// is zero but for rounding, and it is kept: without it a right-hand side near
// breakdown lost its way (7.9e-9 after 2000 iterations at a tolerance of
// 1e-12).
// omega = 0 (t = 0, e.g. s = 0 after an exact half step) ends the recursion:
// beta is set to 0, and the check sends the right-hand side to the FP64 true
// residual, which either confirms convergence or restarts from it.
__device__ __forceinline__ void bicg_omega_step(KState &s, const double d[7])
{
    const double ts[2] = {d[0], d[1]}, tt = d[2], rt[2] = {d[3], d[4]}, rs[2] = {d[5], d[6]};
    if (tt > 0) {
        s.omega[0] = ts[0] / tt;
        s.omega[1] = ts[1] / tt;
    } else {
        s.omega[0] = s.omega[1] = 0.0;
    }
    double wrt[2], rn[2], q[2], ao[2];
    cmul(s.omega, rt, wrt);
    rn[0] = rs[0] - wrt[0];
    rn[1] = rs[1] - wrt[1];
    if (s.omega[0] == 0 && s.omega[1] == 0) {
        s.beta[0] = s.beta[1] = 0.0;
    } else {
        cdiv(rn, s.rho, q);
        cdiv(s.alpha, s.omega, ao);
        cmul(q, ao, s.beta);
    }
    s.rho[0] = rn[0];
    s.rho[1] = rn[1];
}

// After the x / r / p update of an iteration, rr = |r|^2: counts it and flags
// convergence (or the iteration cap, or a breakdown: rho = 0 or omega = 0) for
// the FP64 true-residual check, and a reliable update when |r| fell by delta
// since the last one.
__device__ __forceinline__ void bicg_check_step(KState &s, double rr, double delta2, int maxiter, bool mixed, int &act,
                                                int &upd)
{
    s.iters += 1;
    s.rr = rr;
    if (!isfinite(rr) || !isfinite(s.beta[0]) || !isfinite(s.beta[1])) {
        s.nonfinite = 1;
        act = 0;
        upd = 0;
        return;
    }
    if (rr <= s.stop2 || s.iters >= maxiter || (s.rho[0] == 0 && s.rho[1] == 0) ||
        (s.omega[0] == 0 && s.omega[1] == 0)) {
        // converged (or out of iterations, or breakdown): check the FP64 true residual
        act = 0;
        upd = 1;
    } else if (mixed && rr < delta2 * s.maxrr) {
        upd = 1;
    }
    if (rr > s.maxrr) s.maxrr = rr;
}

// After a reliable update replaced r by the FP64 residual: rn = (rhat, r) of the
// replaced r, which rho takes, so that the next alpha matches the r it
// multiplies (alpha, omega and beta stay); r2 = |r|^2 of the FP64 residual, the
// true residual of the Schur system.
__device__ __forceinline__ void bicg_update_step(KState &s, const double rn[2], double r2, int maxiter, int &act,
                                                 int &restart)
{
    s.rho[0] = rn[0];
    s.rho[1] = rn[1];
    s.true2 = r2;
    s.updates += 1;
    restart = 0;
    if (!isfinite(r2)) {
        s.nonfinite = 1;
        act = 0;
    } else if (r2 <= s.stop2) {
        s.done = 1;
        act = 0;
    } else if (!act && s.iters < maxiter) {
        // the iterated residual claimed convergence but the true one disagrees:
        // restart the recursion from the true residual
        act = 1;
        restart = 1;
    }
    s.maxrr = r2;
    s.rr = r2;
}

}  // namespace dl
