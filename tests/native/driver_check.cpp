// Test infrastructure (CPU): the run driver's planning (driver.hpp) and the
// device's rule for ending a launch (span_plan), run together against the host
// controller taking the same steps one at a time.  The device is played by this
// program: launches run in order on its own controller state, and the host reads
// their records with a random lag, as adpsgd_run does.  Random schedules: every
// period mode, launch policy, warm-up prefixes, period switches, plain and traced,
// 1 to 16 measurements a launch, both kernels (K up to 128 and above), runs cut
// anywhere.  Checked beside the schedule: the rows are read as merged exactly when
// the launch before left them so, and are whole at the end of every run; a launch
// stays within its steps, rates and record slots.  Prints "all ok" at the end.
#include <cstdint>
#include <cstdio>
#include <deque>
#include <random>
#include <vector>

#include "adpsgd.h"
#include "common.hpp"
#include "driver.hpp"

using namespace adpsgd;

namespace adpsgd {   // (runtime.cpp's, which this program does without)
int fail(int code, const std::string &) { return code; }
int ok() { return ADPSGD_OK; }
}  // namespace adpsgd

#define CHECK(cond, ...)                                                    \
    do {                                                                    \
        if (!(cond)) {                                                      \
            std::printf("schedule %d: %s: ", g_case, #cond);                \
            std::printf(__VA_ARGS__);                                       \
            std::printf("\n");                                              \
            return 1;                                                       \
        }                                                                   \
    } while (0)

static int g_case = 0;

struct Sync {
    int64_t t;
    int32_t p;
};

// The variance after step t: any function of t alone will do.
static double variance(const adpsgd_hparams &hp, int64_t t, int drift) {
    uint64_t v = (uint64_t)t * 0x9E3779B97F4A7C15u + hp.seed;
    v ^= v >> 29;
    v *= 0xBF58476D1CE4E5B9u;
    v ^= v >> 32;
    const double u = (double)(v % 1000) / 1000.0;   // the bands are 0.7 and 1.3 of the mean
    return adpsgd_lr(&hp, t) * (drift > 0 ? 0.3 * u : drift < 0 ? 1.5 + u : 2.0 * u) * (t < hp.k_s ? 0.0 : 1.0) +
           adpsgd_lr(&hp, t) * (t < hp.k_s ? 1.0 : 0.0);
}

struct Launch {
    SpanWhen w;
    int n_slots;
    int32_t n;                        // as its record says (device) or as planned
    std::vector<double> S;            // of its measurements
};

struct Counts {
    int64_t launches, device, merged, waits, steps;
};

static int run_case(const adpsgd_hparams &hp, const std::vector<int64_t> &cuts, Planner pl, int drift,
                    std::mt19937_64 &rng, Counts *n) {
    constexpr int kRing = 32, kMaxInflight = 64;
    const SchedRule rule = pl.rule;
    const bool control = rule.period_mode == ADPSGD_PERIOD_ADAPTIVE || pl.by_step;
    adpsgd_state known, ref;
    if (adpsgd_sched_init(&hp, &known) || adpsgd_sched_init(&hp, &ref)) return 1;
    std::vector<Sync> got, want;
    for (int64_t steps : cuts) {
        const int64_t end = known.t + steps;
        pl.end = end;
        while (ref.t < end) {
            const int64_t t = ref.t;
            int32_t due = 0;
            if (adpsgd_sched_step(&hp, &ref, &due)) return 1;
            if (!due) continue;
            want.push_back(Sync{t, ref.p});
            if (adpsgd_sched_on_sync(&hp, &ref, t, variance(hp, t, drift), nullptr)) return 1;
        }
        SchedState dev{known.t, known.cnt, known.nC2, known.C2, known.p, 0};
        int64_t t_dev = known.t;        // steps that the launches so far took
        bool rows_merged = false;       // how they left the rows
        std::deque<Launch> inflight;
        int slots_used = 0;
        int64_t launched = 0;
        Planner::Ahead ahead = Planner::known(known);
        auto account = [&](const Launch &l) -> int {
            size_t slot = 0;
            for (int32_t j = 0; j < l.n; ++j) {
                const int64_t t = known.t;
                int32_t due = 0;
                if (adpsgd_sched_step(&hp, &known, &due)) return 1;
                const bool planned_due = l.w.device ? j == l.n - 1 && due : (l.w.syncs >> j) & 1;
                CHECK((due != 0) == planned_due, "step %lld", (long long)t);
                if (!due && !l.w.measure) continue;
                CHECK(slot < l.S.size(), "step %lld", (long long)t);
                const double S = l.S[slot++];
                CHECK(S == variance(hp, t, drift), "step %lld", (long long)t);
                if (!due) continue;
                got.push_back(Sync{t, known.p});
                if (adpsgd_sched_on_sync(&hp, &known, t, S, nullptr)) return 1;
            }
            CHECK(slot == l.S.size(), "%zu records", l.S.size());
            return 0;
        };
        // read the records of launches at the front: a random number of those that have
        // some, at least one with `wait`
        auto drain = [&](bool wait) -> int {
            bool read = false;
            while (!inflight.empty()) {
                const Launch l = inflight.front();
                if (l.n_slots > 0) {
                    if (!(wait && !read) && rng() % 3) break;
                    read = true;
                    slots_used -= l.n_slots;
                }
                inflight.pop_front();
                if (account(l)) return 1;
            }
            if (read) {
                ahead = Planner::known(known);
                for (const Launch &l : inflight) pl.pass(&ahead, l.w);
            }
            return 0;
        };
        for (;;) {
            if (rng() % 4 == 0 && drain(false)) return 1;
            CHECK(ahead.t_hi <= end && ahead.st.t <= t_dev && t_dev <= ahead.t_hi, "%lld of [%lld, %lld]",
                  (long long)t_dev, (long long)ahead.st.t, (long long)ahead.t_hi);
            if (ahead.t_hi >= end) {
                if (inflight.empty()) break;
                if (drain(true)) return 1;
                continue;
            }
            Launch l{};
            bool wait = !pl.next(ahead, launched == 0, &l.w);
            if (!wait) {
                l.n_slots = measurements(l.w);
                wait = slots_used + l.n_slots > kRing || (int)inflight.size() >= kMaxInflight;
            }
            if (wait) {
                ++n->waits;
                bool records = false;
                for (const Launch &q : inflight) records = records || q.n_slots > 0;
                CHECK(records, "nothing in flight to wait for");
                if (drain(true)) return 1;
                continue;
            }
            CHECK(l.w.n >= 1 && l.w.n <= kSpanSteps && l.n_slots <= std::max(pl.n_slots, 1), "%d steps, %d slots", l.w.n,
                  l.n_slots);
            CHECK(control || !l.w.device, "device-ended launch without a controller");
            CHECK(pl.in_registers || !l.w.device || l.w.n == 1, "%d steps", l.w.n);
            // the device takes the launch
            const SpanPlan sp = span_plan(l.w, &dev, rule);
            CHECK(sp.t == t_dev && sp.n >= 0 && sp.n <= l.w.n && sp.t + sp.n <= end, "t %lld n %d", (long long)sp.t, sp.n);
            CHECK(sp.n > 0 || (l.w.device && !l.w.known), "no step");
            CHECK(sp.t - l.w.t + sp.n <= (l.w.device && !l.w.known ? kSpanSteps : l.w.n), "rates");
            if (sp.n > 0) {
                CHECK(sp.merged_in == rows_merged, "t %lld: rows %s", (long long)sp.t, rows_merged ? "merged" : "whole");
                const bool ends_synced = (sp.syncs >> (sp.n - 1)) & 1;
                CHECK(sp.merged_out == (pl.merge && ends_synced && sp.t + sp.n < end), "t %lld", (long long)sp.t);
                rows_merged = sp.merged_out;
            }
            for (int32_t j = 0; j < sp.n; ++j) {
                const bool due = (sp.syncs >> j) & 1;
                if (due || l.w.measure) l.S.push_back(variance(hp, sp.t + j, drift));
                if (due && control) {
                    dev.p = period_at(rule, dev.p, sp.t + j);
                    (void)apply_sync(rule, sp.t + j, adpsgd_lr(&hp, sp.t + j), l.S.back(), &dev, nullptr);
                }
            }
            if (control && l.n_slots > 0) {   // the reduction keeps the state up
                dev.cnt = sp.syncs ? sp.n - (64 - __builtin_clzll(sp.syncs)) : dev.cnt + (sp.t - dev.t) + sp.n;
                dev.t = sp.t + sp.n;
            }
            l.n = sp.n;
            t_dev += sp.n;
            slots_used += l.n_slots;
            pl.pass(&ahead, l.w);
            ++launched;
            ++n->launches;
            n->device += l.w.device;
            n->merged += sp.merged_in;
            n->steps += sp.n;
            inflight.push_back(l);
        }
        CHECK(known.t == end && t_dev == end && !rows_merged, "t %lld", (long long)known.t);
        CHECK(known.cnt == ref.cnt && known.p == ref.p && known.C2 == ref.C2 && known.nC2 == ref.nC2, "state");
    }
    CHECK(got.size() == want.size(), "%zu syncs of %zu", got.size(), want.size());
    for (size_t i = 0; i < got.size(); ++i)
        CHECK(got[i].t == want[i].t && got[i].p == want[i].p, "sync %zu", i);
    return 0;
}

// Behind a decision in flight a K of the loop kernel (above 128) reads the record
// rather than have the device decide a step, unless p is 1 or 2; the period then is
// one launch.
static int check_launches_of_many_workers() {
    g_case = -1;
    adpsgd_hparams hp{};
    hp.sigma = 0.1; hp.h_lo = 0.1; hp.h_hi = 1.0; hp.lr0 = 0.1; hp.total_steps = 1000; hp.thr_lo = 0.7; hp.thr_hi = 1.3;
    hp.period_mode = ADPSGD_PERIOD_ADAPTIVE;
    hp.p_init = 1;
    for (int32_t p : {1, 2, 3, 4, 9, 64})
        for (int policy : {ADPSGD_LAUNCH_HYBRID, ADPSGD_LAUNCH_HOST}) {
            Planner pl{rule_of(&hp), 1000, 16, false, false, policy == ADPSGD_LAUNCH_HOST, false, false};
            adpsgd_state st{};
            st.t = 500;
            st.p = p;
            Planner::Ahead a = Planner::known(st);
            SpanWhen w;
            CHECK(pl.next(a, false, &w) && !w.device && w.n == p && w.syncs == uint64_t(1) << (p - 1), "p %d", p);
            pl.pass(&a, w);
            CHECK(a.p_open && a.st.t == 500 + p && a.st.cnt == 0, "p %d", p);
            const bool more = pl.next(a, false, &w);
            CHECK(more == (p <= 2 && policy == ADPSGD_LAUNCH_HYBRID), "p %d", p);
            CHECK(!more || (w.device && w.known && w.n == 1 && w.t == 500 + p), "p %d", p);
        }
    return 0;
}

int main() {
    if (check_launches_of_many_workers()) return 1;
    std::mt19937_64 rng(11);
    auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
    Counts n{};
    for (g_case = 0; g_case < 20000; ++g_case) {
        adpsgd_hparams hp{};
        hp.seed = rng();
        hp.sigma = 0.1; hp.h_lo = 0.1; hp.h_hi = 1.0; hp.lr0 = 0.1; hp.total_steps = 1000; hp.thr_lo = 0.7; hp.thr_hi = 1.3;
        hp.period_mode = pick(0, 1) ? ADPSGD_PERIOD_ADAPTIVE : (int32_t)pick(0, 2);
        hp.p_init = (int32_t)pick(1, g_case % 4 == 0 ? 140 : 9);
        hp.p_max = pick(0, 3) == 0 ? hp.p_init + (int32_t)pick(0, 3) : 0;
        hp.k_s = pick(0, 2) == 0 ? 0 : pick(0, 60);
        hp.sync_warmup_steps = pick(0, 3) == 0 ? pick(0, 30) : 0;
        if (hp.period_mode != ADPSGD_PERIOD_ADAPTIVE && pick(0, 1)) {
            hp.p_switch_step = pick(1, 200);
            hp.p_after = (int32_t)pick(1, hp.p_max ? hp.p_max : 9);
        }
        std::string why;
        if (!hparams_valid(&hp, &why)) { std::printf("bad hparams: %s\n", why.c_str()); return 1; }
        const int policy = (int)pick(0, 2);
        Planner pl{};
        pl.rule = rule_of(&hp);
        const int32_t slots[] = {1, 2, 5, 16};
        pl.n_slots = slots[pick(0, 3)];
        pl.measure = pick(0, 2) == 0;
        pl.by_step = policy == ADPSGD_LAUNCH_DEVICE;
        pl.host_waits = policy == ADPSGD_LAUNCH_HOST;
        pl.in_registers = pick(0, 3) != 0;
        pl.merge = !pl.by_step && pl.in_registers && pick(0, 4) != 0;
        std::vector<int64_t> cuts;
        for (int64_t i = pick(1, 4); i > 0; --i) cuts.push_back(pick(0, g_case % 3 ? 90 : 400));
        if (run_case(hp, cuts, pl, (int)pick(-1, 1), rng, &n)) return 1;
    }
    std::printf("%lld launches of %lld steps, %lld ended by the device, %lld with merged rows, %lld waits\nall ok\n",
                (long long)n.launches, (long long)n.steps, (long long)n.device, (long long)n.merged, (long long)n.waits);
    return 0;
}
