// Device side of the solvers' scalar steps: the finalize of a reduction runs
// the step of solver_ctl.h on the grand totals, and kernels test their
// predicate on the control block at the top.  Keeping the scalars on the
// device lets a whole iteration run without a host round trip.
#pragma once

#include "lqcd.h"
#include "lqcd_kernels.h"
#include "solver_ctl.h"

namespace lqcd {

// ctl_step by one wavefront (every lane holds the totals): lane 0, or for the
// multi-shift steps one lane per shift (eight shifts in one lane took 2.5 us
// longer).  The lanes run in step, so all have read the base system before its
// own lane changes it.
__device__ inline void ctl_step_wave(Ctl* c, int pre, const double* pv, int fin, const double* v,
                                     bool always = false)
{
    static_assert(kMaxShifts <= 64, "one lane per shift");
    const int lane = threadIdx.x;
    if (fin != FIN_MS_ALPHA && fin != FIN_MS_BETA) {
        if (lane == 0) ctl_step(c, pre, pv, fin, v, always);
        return;
    }
    const int n = c->ms_n, mine = c->ms_index;
    const bool open = always || !c->done;
    Ctl* ci = c - mine + (lane < n ? lane : mine);
    if (fin == FIN_MS_ALPHA) {
        const MsAlpha m = ms_alpha(c, v[1]);
        __builtin_amdgcn_wave_barrier();
        if (!open || lane >= n) return;
        ms_alpha_shift(ci, m);
        if (lane == mine) c->alpha = m.al;
    } else {
        const MsBeta m = ms_beta(c, v[0]);
        __builtin_amdgcn_wave_barrier();
        if (lane >= n) return;
        if (open) {
            ms_beta_shift(ci, m);
            if (lane == mine) ms_beta_base(c, m);
        }
        ctl_close(ci);
    }
}

__device__ inline bool pred_skip(int pred, const Ctl* c)
{
    if (pred == PRED_ALWAYS || c == nullptr) return false;
    const int done = __hip_atomic_load(&c->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (done) return true;
    if (pred == PRED_UPDATE) return c->update == 0;
    if (pred == PRED_NO_UPDATE) return c->update != 0;
    return false;
}

}  // namespace lqcd
