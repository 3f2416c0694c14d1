// Test infrastructure (CPU): the rule by which the device ends a launch
// (span_plan) against the host controller (adpsgd_sched_*), step by step, over
// random schedules: every period mode, warm-up prefixes, period switches,
// launches with a known and an unknown first step, cut by their most steps, by
// their rates and by the end of the run.  Prints "all ok" at the end.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <random>

#include "adpsgd.h"
#include "common.hpp"
#include "schedule.hpp"

using namespace adpsgd;

namespace adpsgd {   // (runtime.cpp's, which this program does without)
int fail(int code, const std::string &) { return code; }
int ok() { return ADPSGD_OK; }
}  // namespace adpsgd

int main() {
    std::mt19937_64 rng(7);
    auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
    int64_t launches = 0, cut = 0, empty = 0;
    for (int i = 0; i < 4000; ++i) {
        adpsgd_hparams hp{};
        hp.sigma = 0.1; hp.h_lo = 0.1; hp.h_hi = 1.0; hp.lr0 = 0.1; hp.total_steps = 1000; hp.thr_lo = 0.7; hp.thr_hi = 1.3;
        hp.period_mode = (int32_t)pick(0, 2);
        hp.p_init = (int32_t)pick(1, i % 3 == 0 ? 100 : 9);
        hp.p_max = pick(0, 3) == 0 ? hp.p_init + (int32_t)pick(0, 3) : 0;
        hp.k_s = pick(0, 100);
        hp.sync_warmup_steps = pick(0, 2) == 0 ? pick(0, 30) : 0;
        if (hp.period_mode != ADPSGD_PERIOD_ADAPTIVE && pick(0, 1)) {
            hp.p_switch_step = pick(1, 200);
            hp.p_after = (int32_t)pick(1, hp.p_max ? hp.p_max : 9);
        }
        std::string why;
        if (!hparams_valid(&hp, &why)) { std::printf("bad hparams: %s\n", why.c_str()); return 1; }
        const SchedRule rule = rule_of(&hp);
        adpsgd_state st;
        if (adpsgd_sched_init(&hp, &st)) return 1;
        const int64_t end = pick(1, 400);
        SchedState dev{0, 0, 0, 0.0, hp.p_init, 0};   // as the reduction keeps it
        while (st.t < end) {
            // plain steps that the device's state does not follow, before some known starts
            const bool known = pick(0, 1);
            if (known && pick(0, 2) == 0) {
                adpsgd_state next = st;
                int32_t due = 0;
                if (adpsgd_sched_step(&hp, &next, &due)) return 1;
                if (!due) st = next;
                if (st.t >= end) break;
            }
            SpanWhen w{};
            const int64_t lag = known || dev.t != st.t ? 0 : std::min<int64_t>(pick(0, 80), st.t);
            w.known = known || dev.t != st.t;
            w.t = st.t - lag;
            w.end = end;
            w.n = (int32_t)pick(1, kSpanSteps);
            w.device = 1;
            const SpanPlan sp = span_plan(w, &dev, rule);
            int64_t most = std::min<int64_t>(std::min<int64_t>(w.n, kSpanSteps - lag), end - st.t);
            if (sp.t != st.t || sp.n > std::max<int64_t>(most, 0)) { std::printf("start or length: %d\n", i); return 1; }
            ++launches;
            if (sp.n == 0) { ++empty; if (most > 0) return 1; w.known = 1; st.t = st.t; if (lag >= kSpanSteps) continue; return 1; }
            bool synced = false;
            for (int32_t j = 0; j < sp.n; ++j) {
                int32_t due = 0;
                if (adpsgd_sched_step(&hp, &st, &due)) return 1;
                if ((due != 0) != (((sp.syncs >> j) & 1) != 0) || (due && j != sp.n - 1)) {
                    std::printf("sync at step %lld of schedule %d\n", (long long)(st.t - 1), i);
                    return 1;
                }
                if (due) {
                    synced = true;
                    const int64_t t = st.t - 1;
                    const double S = adpsgd_lr(&hp, t) * (double)pick(1, 300) / 100.0;
                    dev.p = period_at(rule, dev.p, t);
                    (void)apply_sync(rule, t, adpsgd_lr(&hp, t), S, &dev, nullptr);
                    if (adpsgd_sched_on_sync(&hp, &st, t, S, nullptr)) return 1;
                }
            }
            if (!synced) {
                ++cut;
                if (sp.n != most) { std::printf("ended early: schedule %d\n", i); return 1; }
                dev.cnt += st.t - dev.t;
            }
            dev.t = st.t;
            if (dev.cnt != st.cnt || (synced && dev.p != st.p) || dev.C2 != st.C2) { std::printf("state: schedule %d\n", i); return 1; }
        }
    }
    std::printf("%lld launches, %lld cut, %lld empty\nall ok\n", (long long)launches, (long long)cut, (long long)empty);
    return 0;
}
