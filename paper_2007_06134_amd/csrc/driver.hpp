// The planning of adpsgd_run's launches, on the host alone: which steps the next
// launch takes, which of them a sync follows, and when a record has to be read
// first.  No device call here, so the whole driver is tested without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>

#include "adpsgd.h"
#include "schedule.hpp"

namespace adpsgd {

// Launches in flight whose end only the device knows, at most: with one queued
// behind the one that runs, the GPU does not wait for the host to read a record;
// more keep it busy where a launch is shorter than that takes.
constexpr int kMaxOpen = 3;

// A span the host planned: steps t .. t + n - 1, bit j of syncs set when a sync
// follows step t + j; measure: every step is measured.
inline SpanWhen planned(int64_t t, int32_t n, uint64_t syncs, bool measure) {
    return SpanWhen{t, t + n, syncs, n, 0, 1, measure ? 1 : 0, 0, 0};
}
inline int measurements(const SpanWhen &w) {
    if (w.measure) return w.n;
    return w.device ? 1 : __builtin_popcountll(w.syncs);
}

// Step st->t of a known schedule: true if a sync follows it (the counter then
// restarts; p stays, whatever the sync decides).
inline bool plan_step(const SchedRule &rule, adpsgd_state *st) {
    const int64_t t = st->t++;
    st->cnt += 1;
    st->p = period_at(rule, st->p, t);
    const bool due = sync_due(rule, st->cnt, st->p, t);
    if (due) st->cnt = 0;
    return due;
}

struct Planner {
    SchedRule rule;
    int64_t end;          // of the run
    int32_t n_slots;      // measurements of one launch at most
    bool measure;         // every step is measured (a traced run)
    bool by_step;         // one step at a time, decided by the device
    bool host_waits;      // the host waits for every decision it needs
    bool in_registers;    // a launch may take several steps and syncs (K up to 128)
    bool merge;           // launches that end with a sync leave merged rows

    // The schedule after every launch in flight, as far as the host knows it: st
    // exactly; exactly but for p, which a decision in flight may move by one
    // (p_open); or only that the next step lies in [st.t, t_hi], behind n_open
    // launches that the device ends after decisions in flight.
    struct Ahead {
        adpsgd_state st;
        int64_t t_hi;
        bool p_open;
        int n_open;
    };
    static Ahead known(const adpsgd_state &st) { return Ahead{st, st.t, false, 0}; }

    // The next launch of a schedule known from state st on: steps up to the most of
    // a launch and `end`, ending after the last sync that fits n_slots (every step needs
    // a slot when all are measured), after a sync whose outcome may move p, or at the
    // end.  Without measurements it is plain steps.  st is moved to the state after it.
    // merged: the rows are merged at its start.
    SpanWhen span(adpsgd_state *st, bool merged) const {
        SpanWhen w = planned(st->t, 0, 0, measure);
        w.end = end;
        w.merge = merge ? 1 : 0;
        w.merged = merged ? 1 : 0;
        int slots = 0;
        adpsgd_state after_sync = *st;   // the state after the last sync of the span
        int32_t n_sync = 0;
        while (w.n < kSpanSteps && st->t < end && slots < n_slots) {
            const int64_t t = st->t;
            const bool due = plan_step(rule, st);
            if (due) w.syncs |= uint64_t(1) << w.n;
            ++w.n;
            if (due || measure) ++slots;
            if (due) {
                after_sync = *st;
                n_sync = w.n;
            }
            if (due && sync_decisive(rule, t)) break;
        }
        // the steps after the last sync go with the next launch, which measures them
        // too, unless the run ends here
        if (n_sync > 0 && st->t < end && !measure) {
            *st = after_sync;
            w.n = n_sync;
        }
        return w;
    }

    // `a` moved past launch w.
    void pass(Ahead *a, const SpanWhen &w) const {
        if (by_step) {
            a->t_hi = ++a->st.t;
        } else if (w.device && (a->p_open || a->n_open > 0)) {
            a->n_open += 1;
            a->t_hi = std::min(end, a->t_hi + w.n);
        } else {
            for (int32_t j = 0; j < w.n && a->st.t < end; ++j) {
                const int64_t t = a->st.t;
                const bool due = plan_step(rule, &a->st);
                a->p_open = a->p_open || (due && sync_decisive(rule, t));
                if (due && w.device) break;
            }
            a->t_hi = a->st.t;
        }
    }

    // The launch that follows those in flight (a, which has not reached the end);
    // false if a record has to be read first.  first: nothing of the run has been
    // launched (the rows are then the caller's, whole).
    bool next(const Ahead &a, bool first, SpanWhen *w) const {
        const adpsgd_state &pl = a.st;
        if (by_step) {
            *w = SpanWhen{pl.t, end, 0, 1, 1, 1, measure ? 1 : 0, 0, 0};
            return true;
        }
        if (!a.p_open && a.n_open == 0) {
            adpsgd_state to = pl;
            *w = span(&to, merge && !first && pl.cnt == 0);
            return true;
        }
        // With too many workers for one launch of a period the device decides a step at a
        // time, each a launch with a reduction, and ends no period early.  With p > 2 at
        // least one step is plain whatever the decision in flight says: read its record,
        // and the whole period goes out as one launch of plain steps and one with its
        // sync.  160 adaptive steps, p = 4, with one device-decided step and then a wait
        // / so: 12.8 / 9.1 ms at K = 200, P = 20,000, 13.6 / 9.9 at K = 150, P = 100,000;
        // with the plain steps queued ahead of the record, in a launch of their own, 9.2
        // and 11.2.  With p of 1 or 2 the device decides: there is little to gain by waiting.
        if (!in_registers && !measure && a.n_open == 0 && pl.p > 2) return false;
        if (host_waits || a.n_open >= kMaxOpen) return false;
        // a span the device ends, of at most as many steps as the longest period
        // that the decisions in flight allow
        const bool at_t = a.n_open == 0;
        const int64_t p_hi = std::min<int64_t>(rule.p_max, (int64_t)pl.p + 1 + a.n_open);
        int64_t most = std::max<int64_t>(1, p_hi - (at_t ? pl.cnt : 0));
        most = std::min(most, end - pl.t);
        if (measure) most = std::min<int64_t>(most, n_slots);
        if (!in_registers) {
            if (!at_t) return false;
            most = 1;
        }
        if (at_t) most = std::min<int64_t>(most, kSpanSteps);
        else if (a.t_hi - pl.t + most > kSpanSteps) return false;   // the rates it may need do not fit
        *w = SpanWhen{pl.t, end, 0, (int32_t)std::min<int64_t>(most, kSpanSteps), 1, at_t ? 1 : 0, measure ? 1 : 0,
                      merge ? 1 : 0, 0};
        return true;
    }
};

}  // namespace adpsgd
