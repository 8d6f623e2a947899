// What the step's kernels share: a system's decisions after its product and
// after its update, and the forms of its sums.

#pragma once

#include "batch_internal.hpp"
#include "wave_ops.hpp"

#include <cmath>

namespace mpcg {
namespace batch {

template <typename T> __device__ inline T fma_b(T a, T b, T c);
template <> __device__ inline float fma_b<float>(float a, float b, float c) { return fmaf(a, b, c); }
template <> __device__ inline double fma_b<double>(double a, double b, double c) { return fma(a, b, c); }

// A partial of an FP32-phase dot product in the precision dot_acc asks for:
// the lane's term (exact in FP64, one rounding in FP32) summed over the wave.
__device__ inline double wave_dot32(bool f32, float x, float y)
{
    return f32 ? (double)wave_dot(x, y) : wave_dot((double)x, (double)y);
}

// What a wave of a step needs of its system, in scalar registers.
struct StepSys {
    int32_t mode, ph_it, src, snap_ci, snap_mask;
    double alpha, beta;
    int32_t split, ds, row0, slice0, nslices;
    int64_t entry0;
    unsigned long long doffs;
};
// live: the fields of the recurrence; at: those set at admission.
__device__ inline StepSys step_sys_of(const BSys &live, const BSys &at)
{
    auto sc = [](int32_t v) { return (int32_t)__builtin_amdgcn_readfirstlane(v); };
    StepSys s;
    s.mode = sc(live.mode);
    s.ph_it = sc(live.ph_it);
    s.src = sc(live.src);
    s.snap_ci = sc(live.snap_ci);
    s.snap_mask = sc(live.snap_mask);
    s.alpha = live.alpha;
    s.beta = live.beta;
    s.split = at.split;
    s.ds = at.ds;
    s.row0 = at.row0;
    s.slice0 = at.slice0;
    s.nslices = at.nslices;
    s.entry0 = at.entry0;
    s.doffs = at.doffs;
    return s;
}

// One thread, v: the sum of the product's partials (d.q, or the squared
// residual of a restart or final check).
__device__ inline void step_product_done(BSys &S, int mode, double v)
{
    const double sb = sqrt(S.bb);
    if (mode == kCg32 || mode == kCg64) {
        const double delta = v;
        S.delta = delta;
        if (!isfinite(delta) || !(delta > 0.0)) {
            if (mode == kCg32 && S.auto_eps && !S.eps_set && S.k0_used != 0) {
                // run-ahead: where the FP32 phase stops depends on eps1
                S.ra_stop = kRaBreakdown;
                S.mode = kHold;
                return;
            }
            if (mode == kCg32) {
                S.flags |= MPCG_FLAG_FP32_BREAKDOWN;
                if (S.auto_eps && !S.eps_set && S.k0_used == 0) S.k0_used = S.n1 < S.k0 ? S.n1 : S.k0;
                S.relres_sp = sqrt(S.gamma) / sb;
                S.src = kSrcX32;
                S.ph_it = 0;
                S.mode = kRestart;
            } else {
                S.pend = isfinite(delta) ? MPCG_ENOTSPD : MPCG_ENONFINITE;
                S.mode = kResid;
            }
            return;
        }
        S.alpha = mode == kCg32 ? (double)(float)(S.gamma / delta) : S.gamma / delta;
        S.upd = 1;
    } else if (mode == kRestart) {
        S.gamma = v;
        S.relres_restart = sqrt(v) / sb;
        S.ph_it = 0;
        if (sqrt(v) <= S.thr2) {
            S.mode = kResid;
        } else if (S.n2 >= S.maxit2) {
            S.pend = MPCG_ENOCONV;
            S.mode = kResid;
        } else {
            S.mode = kCg64;
        }
    } else {   // final check
        const double rho = sqrt(v);
        S.relres_final = rho / sb;
        if (S.pend) {
            S.status = S.pend;
            S.mode = kDone;
        } else if (rho <= S.thr2) {
            S.status = MPCG_OK;
            S.mode = kDone;
        } else if (S.restarts < S.max_restarts) {
            S.restarts += 1;
            S.flags |= MPCG_FLAG_FINAL_RESTARTED;
            S.src = kSrcX64;
            S.mode = kRestart;
        } else {
            S.status = MPCG_ENOCONV;
            S.mode = kDone;
        }
    }
}

// One thread, g: the sum of the update's partials (r.r); hold: more systems
// share the steps than may run ahead of their eps1.
__device__ inline void step_update_done(BSys &S, bool hold, double g)
{
    S.upd = 0;
    const double gp = S.gamma;
    S.gamma_prev = gp;
    S.gamma = g;
    S.ph_it += 1;
    const double sb = sqrt(S.bb);
    if (S.mode == kCg32) {
        S.n1 += 1;
        const bool prefix = S.auto_eps && S.k0_used == 0;
        if (prefix && S.n1 <= S.k0 && S.n1 <= kK0Max) S.ratios[S.n1 - 1] = sqrt(g) / sqrt(gp);
        S.beta = (double)(float)(g / gp);
        if (prefix && (S.n1 >= S.k0 || g == 0.0)) S.k0_used = S.n1;
        if (prefix && S.n1 < S.k0 && g != 0.0) return;   // Algorithm II: k0 iterations first
        if (S.auto_eps && !S.eps_set) {
            // until eps1 is known: record the first crossing of each
            // candidate (x~ is copied by the next product); then either hold
            // (hold: many systems listed) or run ahead
            const double rg = sqrt(g);
            int due = 0, left = 0;
            for (int t = 0; t < kNumEps; ++t) {
                if (S.cross_iter[t] >= 0) continue;
                if (rg <= S.spec_thr[t]) {
                    S.cross_iter[t] = S.n1;
                    S.cross_gamma[t] = g;
                    due |= 1 << t;
                } else {
                    ++left;
                }
            }
            S.snap_mask = due;
            if (hold) {
                // Until the loosest candidate is crossed every choice of eps1
                // needs these iterations; from the first crossing on they may
                // be wasted, so the system waits there for eps1 without taking
                // bandwidth from the others (no iteration past the chosen
                // eps1, no speculative FP64 phase that the choice may
                // discard).  k_set_eps resumes it from the state the
                // sequential method stops in, as after a run-ahead.
                if (due) {
                    S.ra_stop = left == 0 ? kRaAllCrossed : kRaWait;
                    S.mode = kHold;
                } else if (S.n1 >= S.maxit1) {
                    S.ra_stop = kRaMaxit;
                    S.mode = kHold;
                }
            } else if (left == 0) {
                // every candidate crossed before eps1 is known: the FP64 phase
                // starts now from the tightest candidate's state (x~ of this
                // iteration); k_set_eps keeps it when the chosen candidate
                // crossed at this same iteration, else restarts the FP64 phase
                // from the chosen candidate's copy -- the sequential method's
                // state either way
                S.ra_stop = kRaAllCrossed;
                S.spec = 1;
                S.relres_sp = sqrt(g) / sb;
                S.src = kSrcX32;
                S.ph_it = 0;
                S.mode = kRestart;
            } else if (S.n1 >= S.maxit1) {
                S.ra_stop = kRaMaxit;
                S.mode = kHold;
            }
            return;
        }
        if (sqrt(g) <= S.thr1 || S.n1 >= S.maxit1) {
            if (!(sqrt(g) <= S.thr1)) S.flags |= MPCG_FLAG_FP32_MAXIT;
            S.relres_sp = sqrt(g) / sb;
            S.src = kSrcX32;
            S.ph_it = 0;
            S.mode = kRestart;
        }
    } else {
        S.n2 += 1;
        S.beta = g / gp;
        if (sqrt(g) <= S.thr2) {
            S.mode = kResid;
        } else if (S.n2 >= S.maxit2) {
            S.pend = MPCG_ENOCONV;
            S.mode = kResid;
        }
    }
}

}  // namespace batch
}  // namespace mpcg
