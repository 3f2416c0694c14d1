// Algorithm 2's step counter and period controller as inline functions shared
// by the host controller (adpsgd_sched_step, adpsgd_sched_on_sync) and the
// device reduction kernel, so that a decision taken on the GPU during a run is
// the same fp64 computation, in the same order, as the host's.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "adpsgd.h"

namespace adpsgd {

#define ADPSGD_HD __host__ __device__ __forceinline__

// The hyper-parameters that decide when a sync happens and how p moves.
struct SchedRule {
    int32_t period_mode;     // ADPSGD_PERIOD_*
    int32_t p_after;         // the period from p_switch_step on (constant modes)
    int32_t p_max;           // upper bound on p (>= 1)
    int32_t pad_;
    int64_t k_s;             // syncs after steps t < k_s sample C2
    int64_t warmup;          // steps t < warmup sync every step, with no controller update
    int64_t p_switch_step;   // 0: the period never switches
    double thr_lo, thr_hi;   // the bands of Algorithm 2's period decision
};

// Controller state between steps, as in adpsgd_state: t is the next step, cnt
// the steps since the last sync.  On the device it is written only at syncs,
// so the counter after step t' >= t is cnt + (t' - t) + 1.
struct SchedState {
    int64_t t;
    int64_t cnt;
    int64_t nC2;
    double C2;
    int32_t p;
    int32_t pad_;
};

// The period in force at step t: constant modes may switch to p_after
// (Section III-A's two-phase strategies, Section V-B's decreasing period).
ADPSGD_HD int32_t period_at(const SchedRule &r, int32_t p, int64_t t) {
    return (r.period_mode != ADPSGD_PERIOD_ADAPTIVE && r.p_switch_step > 0 && t >= r.p_switch_step) ? r.p_after
                                                                                                   : p;
}

// Does a sync follow step t?  cnt already counts step t (Algorithm 2, lines
// 5 and 8); p is the period in force.  Warm-up steps always sync; Algorithm
// 1's test is t mod p == 0.
ADPSGD_HD bool sync_due(const SchedRule &r, int64_t cnt, int32_t p, int64_t t) {
    if (t < r.warmup) return true;
    if (r.period_mode == ADPSGD_PERIOD_ALG1) return (t % p) == 0;
    return cnt >= p;
}

// Is the sync after step t one whose outcome may move p?
ADPSGD_HD bool sync_decisive(const SchedRule &r, int64_t t) {
    return r.period_mode == ADPSGD_PERIOD_ADAPTIVE && t >= r.k_s && t >= r.warmup;
}

// Algorithm 2's sampling and period decision after the sync that followed
// step t, with S the summed variance and gamma step t's rate: the counter
// restarts; in the sampling phase (t < K_s) C2 becomes the running mean of
// S / gamma; afterwards p moves by one when S leaves
// [thr_lo gamma C2, thr_hi gamma C2] (p within [1, p_max]).  The sync took
// place whatever S is, so the counter restarts in every case; a non-finite S
// then returns false with C2, nC2 and p untouched.
// margin (may be null): signed relative distance of S to the nearer band edge.
ADPSGD_HD bool apply_sync(const SchedRule &r, int64_t t, double gamma, double S, SchedState *st, double *margin) {
    if (margin) *margin = __builtin_nan("");
    st->cnt = 0;
    if (!__builtin_isfinite(S)) return false;
    if (r.period_mode != ADPSGD_PERIOD_ADAPTIVE || t < r.warmup) return true;
    if (t < r.k_s) {
        st->nC2 += 1;
        st->C2 += (S / gamma - st->C2) / (double)st->nC2;
        return true;
    }
    const double lo = r.thr_lo * gamma * st->C2;
    const double hi = r.thr_hi * gamma * st->C2;
    if (margin && lo > 0) {
        const double m_lo = S / lo - 1.0, m_hi = S / hi - 1.0;
        *margin = __builtin_fabs(m_lo) < __builtin_fabs(m_hi) ? m_lo : m_hi;
    }
    if (S < lo) {
        if (st->p < r.p_max) st->p += 1;
    } else if (S > hi) {
        if (st->p > 1) st->p -= 1;
    }
    return true;
}

constexpr int kSpanSteps = 64;   // steps per launch at most

// Which steps a launch takes and which of them a sync follows.  The host plans
// both (device = 0: steps t .. t + n - 1, bit j of syncs set when a sync follows
// step t + j), or the launch ends with the first step that the device's
// controller state says is due, after n steps or before step `end`, whichever
// comes first; it starts at t (known) or at the state's next step, which is then
// at most kSpanSteps - 1 beyond t, the step of the launch's first rate.
//
// Merged rows: behind a sync the K rows of x are equal (and of m, where momentum
// is averaged), so inside a run a launch that ends with a sync writes row 0
// alone and the next one reads row 0 for all.  Every launch with a sync of such
// a run does so (merge), except that the run's last step leaves whole rows.
struct SpanWhen {
    int64_t t;
    int64_t end;       // the run's end
    uint64_t syncs;
    int32_t n;
    int32_t device;
    int32_t known;
    int32_t measure;   // 1: every step is measured, not only those a sync follows
    int32_t merge;     // 1: a sync at the launch's end leaves merged rows
    int32_t merged;    // (host-planned) the rows are merged at the start
};
struct SpanPlan {
    int64_t t;         // the first step
    int32_t n;         // steps (0: nothing is left to do)
    bool merged_in, merged_out;
    uint64_t syncs;
};

// The controller state is the device's at the start of the launch (read by
// every thread, written only by the reduction that follows), so the answer is
// uniform over the launch and its reduction.
ADPSGD_HD SpanPlan span_plan(const SpanWhen &w, const SchedState *sched, const SchedRule &r) {
    SpanPlan p{w.t, w.n, w.merged != 0, false, w.syncs};
    if (w.device) {
        const SchedState s = *sched;
        if (!w.known) p.t = s.t;
        p.n = 0;
        p.syncs = 0;
        int64_t most = w.n < kSpanSteps - (p.t - w.t) ? w.n : kSpanSteps - (p.t - w.t);
        if (most > w.end - p.t) most = w.end - p.t;
        int64_t cnt = s.cnt + (p.t - s.t);
        p.merged_in = w.merge && cnt == 0;   // (a launch of the run ended with the last sync)
        while (p.n < most) {
            const int64_t t = p.t + p.n;
            ++p.n;
            if (sync_due(r, ++cnt, period_at(r, s.p, t), t)) {
                p.syncs = uint64_t(1) << (p.n - 1);
                break;
            }
        }
    }
    p.merged_out = w.merge && p.n > 0 && ((p.syncs >> (p.n - 1)) & 1) && p.t + p.n < w.end;
    return p;
}

#undef ADPSGD_HD

}  // namespace adpsgd
