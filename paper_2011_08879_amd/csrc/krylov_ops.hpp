// The scalar steps of the Krylov recurrences: what one thread does with the
// totals of a reduction.  The finalize kernels of large systems apply them in
// place (on_state); the kernels of mid-size systems apply them to the state
// that they work with (midsize.hip).
#pragma once

#include <cmath>

#include "solver_state.hpp"

namespace gko {

// alpha = rho / p.q; p.q <= 0 means A is not SPD.
struct cg_alpha_step {
    static constexpr int NV = 1;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        const double pq = o[0];
        s.aux = pq;
        if (!(pq > 0.0)) {
            s.done = std::isnan(pq) ? kBreakdown : kNotSpd;
            s.iter += 1;
        } else {
            s.alpha = s.rho / pq;
        }
    }
};

// After the update: totals r.z, r.r (and, for flexible CG, z.(r - r_old));
// convergence test, then beta: r.z / rho (Fletcher-Reeves, CG) or
// z.(r - r_old) / rho (Polak-Ribiere, flexible CG).
struct cg_update_step {
    bool flex;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        s.iter += 1;
        s.half = 1;
        s.rr = o[1];
        if (!std::isfinite(o[1]) || !std::isfinite(o[0])) {
            s.done = kBreakdown;
        } else if (o[1] <= s.stop2) {
            s.done = kConverged;
        } else {
            s.beta = (flex ? o[2] : o[0]) / s.rho;
            s.rho = o[0];
            if (s.iter >= s.maxit) s.done = kMaxIter;
        }
    }
};

// BiCGSTAB: alpha = rho / (rhat.v)
struct bicg_alpha_step {
    static constexpr int NV = 1;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        s.aux = o[0];
        if (!(fabs(o[0]) >= 1e-300)) s.done = kBreakdown;
        else s.alpha = s.rho / o[0];
    }
};

// s.s: converging here finishes at the half step.
struct bicg_s_step {
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        s.iter += 1;
        if (!std::isfinite(o[0])) s.done = kBreakdown;
        else if (o[0] <= s.stop2) {
            s.half = 1;
            s.rr = o[0];
        }
    }
};

// omega = (t.s) / (t.t); nothing at the half step.
struct bicg_omega_step {
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        if (s.half) return;
        s.aux = o[1];
        if (!(o[1] >= 1e-300)) s.done = kBreakdown;
        else s.omega = o[0] / o[1];
    }
};

// After the update: totals r.r and the next rho = rhat.r.
struct bicg_update_step {
    static constexpr int NV = 2;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        if (s.half) {
            s.done = kConverged;
            return;
        }
        s.rr = o[0];
        if (!std::isfinite(o[0])) s.done = kBreakdown;
        else if (o[0] <= s.stop2) s.done = kConverged;
        else if (s.omega == 0.0) s.done = kBreakdown;
        else {
            s.rho_old = s.rho;
            s.rho = o[1];
            if (!(fabs(o[1]) >= 1e-300)) s.done = kBreakdown;
            else {
                s.beta = (s.rho / s.rho_old) * (s.alpha / s.omega);
                if (s.iter >= s.maxit) s.done = kMaxIter;
            }
        }
    }
};

// CGS: alpha = rho / (t.rhat)
struct cgs_alpha_step {
    static constexpr int NV = 1;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        s.aux = o[0];
        if (!(fabs(o[0]) >= 1e-300)) s.done = kBreakdown;
        else s.alpha = s.rho / o[0];
    }
};

// After r -= alpha A (u + q): totals r.r, r.rhat; convergence, then beta.
struct cgs_update_step {
    static constexpr int NV = 2;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        s.iter += 1;
        s.rr = o[0];
        if (!std::isfinite(o[0])) s.done = kBreakdown;
        else if (o[0] <= s.stop2) s.done = kConverged;
        else if (s.iter >= s.maxit) s.done = kMaxIter;
        else if (!(fabs(o[1]) >= 1e-300)) s.done = kBreakdown;
        else {
            s.beta = o[1] / s.rho;
            s.rho = o[1];
        }
    }
};

// Pipelined CG: alpha and beta of the step that follows the sums gamma,
// delta: first step beta = 0, alpha = gamma / delta; then beta = gamma /
// gamma_old, alpha = gamma / (delta - beta gamma / alpha_old).  The
// denominator is p.Ap in exact arithmetic, <= 0 means A is not SPD.
__device__ inline void pipe_next(krylov_scalars &s, double gamma, double delta, bool first) {
    const double beta = first ? 0.0 : gamma / s.rho;
    const double den = first ? delta : delta - beta * gamma / s.alpha;
    s.aux = den;
    if (!(den > 0.0)) {
        s.done = std::isnan(den) ? kBreakdown : kNotSpd;
        s.iter += 1;
        return;
    }
    s.beta = beta;
    s.alpha = gamma / den;
    s.rho = gamma;
}

// After an update: totals gamma, delta, r.r.
struct pipe_update_step {
    static constexpr int NV = 3;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        s.iter += 1;
        s.rr = o[2];
        if (!std::isfinite(o[2]) || !std::isfinite(o[0]) || !std::isfinite(o[1])) s.done = kBreakdown;
        else if (o[2] <= s.stop2) s.done = kConverged;
        else if (s.iter >= s.maxit) s.done = kMaxIter;
        else pipe_next(s, o[0], o[1], false);
    }
};

// A step applied in place to the totals (by the finalize kernel, or by the
// last block of a small grid).
template <typename Step>
struct on_state {
    krylov_scalars *sc;
    Step step;
    __device__ bool skip() const { return sc->done != 0; }
    __device__ void operator()(const double *o) const { step(*sc, o); }
};
using cg_alpha_op = on_state<cg_alpha_step>;
using cg_update_op = on_state<cg_update_step>;
using bicg_alpha_op = on_state<bicg_alpha_step>;
using bicg_s_op = on_state<bicg_s_step>;
using bicg_omega_op = on_state<bicg_omega_step>;
using bicg_update_op = on_state<bicg_update_step>;
using cgs_alpha_op = on_state<cgs_alpha_step>;
using cgs_update_op = on_state<cgs_update_step>;
using pipe_update_op = on_state<pipe_update_step>;

}  // namespace gko
