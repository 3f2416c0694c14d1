// Host runtime and C ABI of the ADPSGD hot path: argument validation, the tile
// table of the segmented variance reduction, kernel launches on the caller's
// stream, the Algorithm 2 driver (host-planned steps, device-decided syncs
// where the host has not yet read a decision back), checkpoint state and
// timing.
#include <hip/hip_runtime.h>

#include <rocprofiler-sdk-roctx/roctx.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <deque>
#include <limits>
#include <mutex>
#include <new>
#include <string>
#include <unordered_set>
#include <vector>

#include "adpsgd.h"
#include "common.hpp"
#include "driver.hpp"
#include "kernels.hpp"

namespace adpsgd {

thread_local std::string g_last_error;

int fail(int code, const std::string &msg) {
    g_last_error = msg;
    return code;
}
int ok() {
    g_last_error.clear();
    return ADPSGD_OK;
}

// Windows of tensors for the second level of the variance sum when there are
// more chunk partials than one LDS window holds: runs of whole small tensors
// (at most kSmallTensorChunks chunks each) whose chunks fit kFinishWindow, and
// every larger tensor alone.  win_begin receives the first tensor of each
// window and T; returns the window count (0, with win_begin empty, when one
// window holds every chunk partial).
int32_t reduce_windows(int32_t T, const int32_t *chunk_begin, std::vector<int32_t> *win_begin) {
    win_begin->clear();
    if (chunk_begin[T] <= kFinishWindow) return 0;
    win_begin->push_back(0);
    int32_t cur = 0;  // chunks in the current run of small tensors
    for (int32_t tau = 0; tau < T; ++tau) {
        const int32_t c = chunk_begin[tau + 1] - chunk_begin[tau];
        if (c > kSmallTensorChunks) {
            if (tau > win_begin->back()) win_begin->push_back(tau);
            win_begin->push_back(tau + 1);
            cur = 0;
        } else if (cur + c > kFinishWindow) {
            win_begin->push_back(tau);
            cur = c;
        } else {
            cur += c;
        }
    }
    if (win_begin->back() < T) win_begin->push_back(T);
    return (int32_t)win_begin->size() - 1;
}

namespace {

constexpr int kRing = 32;          // record slots: launches with a reduction in flight at once
constexpr int kTimedMax = 4096;    // pending timed launches before a harvest
// Measurements (syncs, or steps of a traced run) of one launch at most, and the
// device memory their partial sums may take (one measurement's always fits).
constexpr int32_t kSpanSlots = 16;
constexpr int64_t kSpanSlotBytes = int64_t(64) << 20;
constexpr int64_t kMaxInflight = 64;   // launches the host has not yet accounted for
// Between waits, the driver polls for finished records every kPollEvery launches
// (each poll is a runtime call; steps without a record need no accounting to proceed).
constexpr int64_t kPollEvery = 8;
// adpsgd_init times the local step's block sizes when one step moves at least
// this many elements (below it a launch is too short to time reliably).
constexpr double kTuneMinElems = 16.0 * 1024 * 1024;
// Below the same size a step takes a few microseconds on the GPU, less than
// the host needs to launch it, so runs whose schedule is known in advance
// (the constant-period modes) are captured once as a HIP graph and replayed;
// runs of up to kGraphMaxSteps steps.
constexpr double kGraphMaxElems = kTuneMinElems;
constexpr int64_t kGraphMaxSteps = int64_t(1) << 16;
constexpr int64_t kMaxK = 65536;
constexpr int64_t kMaxCounter = int64_t(1) << 32;  // Philox counter words are 32-bit

enum TimedKind { tStep = 0, tFused = 1, tAverage = 2, tSegsum = 3, tTrace = 4, tKinds = 5 };
// Sampling classes of the timer: the timed kinds, plus the spans, whose steps are
// told apart when they are accounted for.
enum { cSpan = tKinds, kTimedClasses = tKinds + 1 };

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

bool shape_valid(int32_t K, int64_t P, int32_t T, const int64_t *off, std::string *why) {
    auto bad = [&](const std::string &m) { if (why) *why = m; return false; };
    if (K < 1 || K > kMaxK) return bad("K must be in [1, 65536]");
    if (P < 0) return bad("P must be >= 0");
    if ((P + 3) / 4 > kMaxCounter) return bad("P/4 must be below 2^32");
    if (T < 1 || T > (1 << 24)) return bad("T must be in [1, 2^24]");
    if (!off) return bad("tensor_offsets is NULL");
    if (off[0] != 0) return bad("tensor_offsets[0] must be 0");
    for (int32_t i = 0; i < T; ++i)
        if (off[i + 1] < off[i]) return bad("tensor_offsets must be non-decreasing");
    if (off[T] != P) return bad("tensor_offsets[T] must equal P");
    return true;
}

// Tiles: each tensor [a, b) is cut at multiples of kTileElems, so no tile
// crosses a tensor boundary and a tile spans at most kTileElems / 4 groups.
// Chunks: runs of at most chunk_tiles consecutive tiles of one tensor, where
// chunk_tiles is 1 for at most kDirectMaxTiles tiles (the tile partials then
// serve as chunk partials) and kChunkTiles otherwise.
int64_t tiles_of(int64_t a, int64_t b) { return b > a ? (b + kTileElems - 1) / kTileElems - a / kTileElems : 0; }

struct Plan {
    int64_t n_tiles = 0, n_chunks = 0;
    int64_t n_aligned = 0;  // aligned chunks of kTileElems elements (a sync-tile block each)
    int32_t chunk_tiles = kChunkTiles;
    int32_t n_windows = 0;  // windows of tensors for k_reduce_windows (0: none)
    int32_t n_slots = 1;    // measurements whose partial sums the workspace holds
};

Plan count_plan(int32_t T, const int64_t *off) {
    Plan pl;
    for (int32_t tau = 0; tau < T; ++tau) pl.n_tiles += tiles_of(off[tau], off[tau + 1]);
    pl.n_aligned = (off[T] + kTileElems - 1) / kTileElems;
    pl.chunk_tiles = pl.n_tiles <= kDirectMaxTiles ? 1 : kChunkTiles;
    std::vector<int32_t> chunk_begin(T + 1, 0);
    for (int32_t tau = 0; tau < T; ++tau) {
        const int64_t n = (tiles_of(off[tau], off[tau + 1]) + pl.chunk_tiles - 1) / pl.chunk_tiles;
        chunk_begin[tau + 1] = chunk_begin[tau] + (int32_t)n;
        pl.n_chunks += n;
    }
    std::vector<int32_t> win_begin;
    pl.n_windows = reduce_windows(T, chunk_begin.data(), &win_begin);
    const int64_t per_slot = 16 * (pl.n_tiles + pl.n_chunks + T + pl.n_windows);
    pl.n_slots = (int32_t)std::min<int64_t>(kSpanSlots, std::max<int64_t>(1, kSpanSlotBytes / per_slot));
    return pl;
}

void build_plan(int32_t T, const int64_t *off, int32_t chunk_tiles, std::vector<Tile> *tiles,
                std::vector<Chunk> *chunks, std::vector<int32_t> *chunk_begin) {
    tiles->clear();
    chunks->clear();
    chunk_begin->assign(T + 1, 0);
    for (int32_t tau = 0; tau < T; ++tau) {
        (*chunk_begin)[tau] = (int32_t)chunks->size();
        const int32_t first_tile = (int32_t)tiles->size();
        for (int64_t s = off[tau]; s < off[tau + 1];) {
            const int64_t e = std::min(off[tau + 1], (s / kTileElems + 1) * kTileElems);
            tiles->push_back(Tile{s, (int32_t)(e - s), tau});
            s = e;
        }
        const int32_t n = (int32_t)tiles->size() - first_tile;
        for (int32_t c = 0; c < n; c += chunk_tiles)
            chunks->push_back(Chunk{first_tile + c, std::min(chunk_tiles, n - c), tau, 0});
    }
    (*chunk_begin)[T] = (int32_t)chunks->size();
}

struct Layout {
    size_t tiles, chunks, chunk_begin, large, tile_partials, chunk_partials, acc, win_begin, win_partials, sums,
        sched, chunk_seg, total;
};

// A record slot (pinned host memory the reduction writes directly): the
// header, then the T variances and the T gradient norms.
size_t slot_bytes_for(int32_t T) { return align_up(kSlotHdrBytes + 2 * sizeof(double) * (size_t)T, 256); }

Layout layout_for(const Plan &pl, int32_t T) {
    auto at_least_one = [](int64_t n) { return (size_t)std::max<int64_t>(n, 1); };
    const size_t slots = (size_t)pl.n_slots;
    Layout l;
    l.tiles = 0;
    l.chunks = align_up(l.tiles + sizeof(Tile) * at_least_one(pl.n_tiles), 256);
    l.chunk_begin = align_up(l.chunks + sizeof(Chunk) * at_least_one(pl.n_chunks), 256);
    l.large = align_up(l.chunk_begin + sizeof(int32_t) * (size_t)(T + 1), 256);
    l.tile_partials = align_up(l.large + sizeof(int32_t) * (size_t)T, 256);
    l.chunk_partials = align_up(l.tile_partials + slots * 2 * sizeof(double) * at_least_one(pl.n_tiles), 256);
    l.acc = align_up(l.chunk_partials + slots * 2 * sizeof(double) * at_least_one(pl.n_chunks), 256);
    l.win_begin = align_up(l.acc + slots * 2 * sizeof(double) * (size_t)T, 256);
    l.win_partials = align_up(l.win_begin + sizeof(int32_t) * (size_t)(pl.n_windows + 1), 256);
    l.sums = align_up(l.win_partials + slots * 2 * sizeof(double) * at_least_one(pl.n_windows), 256);
    l.sched = align_up(l.sums + slots * 2 * sizeof(double), 256);
    l.chunk_seg = align_up(l.sched + sizeof(SchedState), 256);
    l.total = align_up(l.chunk_seg + sizeof(int32_t) * (size_t)(pl.n_aligned + 1), 256);
    return l;
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

int hip_fail(hipError_t e, const char *what) {
    return fail(ADPSGD_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(expr)                                         \
    do {                                                      \
        hipError_t e_ = (expr);                               \
        if (e_ != hipSuccess) return hip_fail(e_, #expr);     \
    } while (0)

struct TimedLaunch {
    int kind;        // -1: a span that is not accounted for
    hipEvent_t start, stop;
    int32_t steps;   // launches of one step that this one stands for
    int32_t syncs;   // of them, those with a sync (a span's; the others are of `kind`)
};

}  // namespace
}  // namespace adpsgd

using namespace adpsgd;

struct adpsgd_ctx {
    int32_t K = 0;
    int64_t P = 0;
    int64_t ld = 0;                 // row stride of x and m (elements)
    int32_t T = 0;
    std::vector<int64_t> offsets;
    std::vector<Tile> tiles;
    std::vector<Chunk> chunks;
    std::vector<int32_t> chunk_begin;
    std::vector<int32_t> large;     // tensors of more than kSmallTensorChunks chunks
    std::vector<int32_t> win_begin; // windows of tensors for k_reduce_windows (empty: none)
    int32_t *d_win_begin = nullptr;
    double *d_win_partials = nullptr;
    adpsgd_hparams hp{};
    adpsgd_buffers buf{};
    hipStream_t stream = nullptr;
    int device = 0;
    Tile *d_tiles = nullptr;
    Chunk *d_chunks = nullptr;
    int32_t *d_chunk_begin = nullptr;
    int32_t *d_large = nullptr;
    std::vector<int32_t> chunk_seg; // first tile of each aligned chunk (the sync-tile kernel's blocks)
    int32_t *d_chunk_seg = nullptr;
    bool chunks_are_tiles = false;  // every tile is its own chunk (small problems)
    double *d_tile_partials = nullptr;
    double *d_chunk_partials = nullptr;
    double *d_acc = nullptr;        // [n_slots][2T] reduction scratch
    double *d_sums = nullptr;       // [n_slots][2]
    int32_t n_slots = 1;            // measurements of one launch at most
    SchedState *d_sched = nullptr;  // the controller state as the device sees it during a run
    char *h_slots = nullptr;        // [kRing] record slots: pinned, coherent host memory
    char *d_slots = nullptr;        // the same slots as the device addresses them
    SchedState *h_sched = nullptr;  // pinned staging for the device controller state
    size_t slot_bytes = 0;
    hipEvent_t ring_ev[kRing] = {};
    adpsgd_state st{};
    bool vec = true;                // row stride % 4 == 0: rows 16-byte aligned, dwordx4 groups
    bool nontemporal = false;       // stream x and m past the caches (large working sets)
    // the same for spans and for the separate sync, timed at init on large working sets
    bool sync_nt = false;
    bool average_nt = false;
    int32_t policy = ADPSGD_LAUNCH_HYBRID;
    StepShape step_shape{256, 0, 1};   // launch shape of the plain local step in use
    StepShape tuned_shape{256, 0, 1};  // the fastest one measured at init
    int32_t average_cap = 0;        // resident blocks per CU of the separate sync (0: no cap), timed at init
    RoundKeys rk{};
    bool timing = false;
    int32_t timing_every = 1;       // time every n-th launch of each class
    int64_t class_seen[kTimedClasses] = {}, class_timed[kTimedClasses] = {};  // steps since timing was set
    std::deque<TimedLaunch> timed;
    int64_t timed_popped = 0;       // timed launches harvested so far (sequence of timed.front())
    std::vector<hipEvent_t> ev_pool;
    double t_ms[tKinds] = {};
    int64_t t_n[tKinds] = {};
    // A constant-period run captured as a HIP graph (run_impl): captured on a
    // private non-blocking stream, launched on the context's stream, kept for
    // as long as runs repeat with the same start state, length and launch shape.
    hipStream_t cap_stream = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    int64_t graph_key[7] = {};
    int64_t graph_captures = 0, graph_replays = 0;   // since the last adpsgd_set_timing
    char *h_gslots = nullptr;       // one record slot per sync of the captured run (pinned)
    char *d_gslots = nullptr;
    int64_t gslot_cap = 0;
};

namespace {

void drop_graph(adpsgd_ctx *c) {
    if (c->graph_exec) (void)hipGraphExecDestroy(c->graph_exec);
    if (c->graph) (void)hipGraphDestroy(c->graph);
    c->graph_exec = nullptr;
    c->graph = nullptr;
}

void release(adpsgd_ctx *c) {
    if (!c) return;
    drop_graph(c);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    if (c->h_gslots) (void)hipHostFree(c->h_gslots);
    for (auto &ev : c->ring_ev)
        if (ev) (void)hipEventDestroy(ev);
    for (auto &tl : c->timed) {
        (void)hipEventDestroy(tl.start);
        (void)hipEventDestroy(tl.stop);
    }
    for (auto ev : c->ev_pool) (void)hipEventDestroy(ev);
    if (c->h_slots) (void)hipHostFree(c->h_slots);
    if (c->h_sched) (void)hipHostFree(c->h_sched);
    delete c;
}

int pool_event(adpsgd_ctx *c, hipEvent_t *ev) {
    if (!c->ev_pool.empty()) {
        *ev = c->ev_pool.back();
        c->ev_pool.pop_back();
        return ok();
    }
    HIP_TRY(hipEventCreate(ev));
    return ok();
}

// Fold finished timed launches into the totals (all of them if wait_all).  A
// launch whose kind is still open (-1: a span the driver has not accounted
// for) stops a non-waiting harvest.  A span's time is shared evenly by its steps.
int harvest(adpsgd_ctx *c, bool wait_all) {
    while (!c->timed.empty()) {
        TimedLaunch tl = c->timed.front();
        if (wait_all) {
            HIP_TRY(hipEventSynchronize(tl.stop));
        } else {
            if (tl.kind < 0) break;
            hipError_t q = hipEventQuery(tl.stop);
            if (q == hipErrorNotReady) break;
            if (q != hipSuccess) return hip_fail(q, "hipEventQuery");
        }
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, tl.start, tl.stop));
        const int kind = tl.kind < 0 ? tStep : tl.kind;
        const double each = (double)ms / std::max(tl.steps, 1);
        c->t_ms[kind] += each * (tl.steps - tl.syncs);
        c->t_n[kind] += tl.steps - tl.syncs;
        c->t_ms[tFused] += each * tl.syncs;
        c->t_n[tFused] += tl.syncs;
        c->ev_pool.push_back(tl.start);
        c->ev_pool.push_back(tl.stop);
        c->timed.pop_front();
        ++c->timed_popped;
    }
    return ok();
}

// Launch, with HIP events around it when timing is on and this launch is
// sampled: a launch of `steps` steps counts as that many of its class.  The first
// launch of a class is timed (work of fewer than timing_every launches' steps
// would go unseen otherwise), then one with which no more than one in
// timing_every of the class (rounded up) is timed.  kind -1: a span, described later (set_span).  *seq (may
// be null) receives the launch's sequence number, or -1 when it is not timed.
template <class F>
int timed_launch(adpsgd_ctx *c, int kind, F launch, int64_t *seq = nullptr, int32_t steps = 1) {
    if (seq) *seq = -1;
    const int cls = kind < 0 ? cSpan : kind;
    bool sampled = false;
    if (c->timing) {
        c->class_seen[cls] += steps;
        sampled = c->class_timed[cls] == 0 ||
                  (c->class_timed[cls] + steps) * c->timing_every <= c->class_seen[cls] + c->timing_every - 1;
    }
    if (!sampled) {
        HIP_TRY(launch());
        return ok();
    }
    c->class_timed[cls] += steps;
    if ((int)c->timed.size() >= kTimedMax) {
        int rc = harvest(c, false);
        if (rc) return rc;
        if ((int)c->timed.size() >= kTimedMax) {
            rc = harvest(c, true);
            if (rc) return rc;
        }
    }
    TimedLaunch tl{kind, nullptr, nullptr, steps, 0};
    int rc = pool_event(c, &tl.start);
    if (rc) return rc;
    rc = pool_event(c, &tl.stop);
    if (rc) return rc;
    HIP_TRY(hipEventRecord(tl.start, c->stream));
    HIP_TRY(launch());
    HIP_TRY(hipEventRecord(tl.stop, c->stream));
    if (seq) *seq = c->timed_popped + (int64_t)c->timed.size();
    c->timed.push_back(tl);
    return ok();
}

// A span of at most `most` steps (timed under sequence number seq, or not) took n,
// `syncs` of them with a sync and the others of `kind`.
void set_span(adpsgd_ctx *c, int64_t seq, int32_t most, int kind, int32_t n, int32_t syncs) {
    if (c->timing) c->class_seen[cSpan] += n - most;   // (the sampling counted the most)
    const int64_t i = seq - c->timed_popped;
    if (seq < 0 || i < 0 || i >= (int64_t)c->timed.size()) return;
    TimedLaunch &tl = c->timed[(size_t)i];
    c->class_timed[cSpan] += n - tl.steps;
    tl.kind = kind;
    tl.steps = n;
    tl.syncs = syncs;
}

StepParams step_params(const adpsgd_ctx *c, int64_t t, int32_t n = 1) {
    StepParams p;
    p.x = c->buf.x;
    p.m = c->buf.m;
    p.h = c->buf.h;
    p.xs = c->buf.xstar;
    p.ld = c->ld;
    p.P = c->P;
    p.n_groups = (c->P + 3) / 4;
    p.K = c->K;
    p.t = (uint32_t)t;
    p.sigma_r = (float)(c->hp.sigma * std::sqrt(2.0 * M_LN2));
    p.mu = (float)c->hp.momentum;
    p.wd = (float)c->hp.weight_decay;
    p.n = n;
    for (int32_t j = 0; j < n; ++j) p.gamma[j] = (float)adpsgd_lr(&c->hp, t + j);
    p.rk = c->rk;
    p.row_chunks = 1;  // set by launch_local_step from the launch shape
    p.block0 = 0;
    return p;
}

// Steps t0 .. t0 + n - 1, up to kSpanSteps of them per launch.
int enqueue_steps(adpsgd_ctx *c, int64_t t0, int64_t n) {
    for (int64_t j = 0; j < n; j += kSpanSteps) {
        const int32_t m = (int32_t)std::min<int64_t>(kSpanSteps, n - j);
        const StepParams p = step_params(c, t0 + j, m);
        int rc = timed_launch(
            c, tStep, [&] { return launch_local_step(p, c->vec, c->nontemporal, c->step_shape, c->stream); }, nullptr, m);
        if (rc) return rc;
    }
    return ok();
}

SyncParams sync_params(const adpsgd_ctx *c) {
    SyncParams sp;
    sp.s = step_params(c, 0);
    sp.tiles = c->d_tiles;
    sp.partials = c->d_tile_partials;
    sp.chunk_seg = c->d_chunk_seg;
    sp.n_chunks = (int64_t)c->chunk_seg.size() - 1;
    return sp;
}

// Rates from step w.t on: a launch with an unknown first step may begin up to
// kSpanSteps - 1 steps later.
int32_t n_rates(const SpanWhen &w) { return w.device && !w.known ? kSpanSteps : w.n; }

SpanParams span_params(const adpsgd_ctx *c, const SpanWhen &w) {
    SpanParams sp;
    static_cast<SyncParams &>(sp) = sync_params(c);
    sp.s = step_params(c, w.t, n_rates(w));
    sp.slot_stride = 2 * (int64_t)c->tiles.size();
    sp.sched = c->d_sched;
    sp.rule = rule_of(&c->hp);
    sp.when = w;
    sp.avg_m = c->hp.avg_momentum;
    sp.pad_ = 0;
    return sp;
}

hipError_t launch_span_of(const adpsgd_ctx *c, const SpanWhen &w, bool nt, hipStream_t st) {
    return launch_span(span_params(c, w), (int64_t)c->tiles.size(), c->vec, nt, c->nontemporal, c->step_shape, st);
}

const char *slot_host(const adpsgd_ctx *c, int slot) { return c->h_slots + (size_t)slot * c->slot_bytes; }

// The reduction of a launch's measurements, their records written from slot
// `slot0` on of the ring at device address recs (with the controller on the
// device when control).
ReduceParams reduce_params(const adpsgd_ctx *c, const SpanWhen &w, char *recs, int slot0, int ring, bool control) {
    ReduceParams r;
    r.tile_partials = c->d_tile_partials;
    r.chunks = c->d_chunks;
    r.chunk_begin = c->d_chunk_begin;
    r.chunk_partials = c->chunks_are_tiles ? c->d_tile_partials : c->d_chunk_partials;
    r.tile_stride = 2 * (int64_t)c->tiles.size();
    r.chunk_stride = 2 * (int64_t)c->chunks.size();
    r.chunks_are_tiles = c->chunks_are_tiles ? 1 : 0;
    r.block0 = 0;
    r.acc = c->d_acc;
    r.sums = c->d_sums;
    r.n_chunks = (int32_t)c->chunks.size();
    r.T = c->T;
    r.K = c->K;
    r.large = c->d_large;
    r.n_large = (int32_t)c->large.size();
    r.win_begin = c->d_win_begin;
    r.win_partials = c->d_win_partials;
    r.n_windows = c->win_begin.empty() ? 0 : (int32_t)c->win_begin.size() - 1;
    r.n_slots = measurements(w);
    r.recs = recs;
    r.slot_bytes = (int64_t)c->slot_bytes;
    r.slot0 = slot0;
    r.ring = ring;
    r.sched = c->d_sched;
    r.control = control ? 1 : 0;
    r.pad_ = 0;
    r.rule = rule_of(&c->hp);
    r.when = w;
    for (int32_t j = 0; j < n_rates(w); ++j) r.gamma[j] = adpsgd_lr(&c->hp, w.t + j);
    return r;
}

// Sync now, without a step (average) or after step t: the kernel, then the
// reduction into record slot 0, then that slot's event.
int enqueue_sync(adpsgd_ctx *c, bool average, int64_t t) {
    const SpanWhen w = planned(t, 1, 1, false);
    int rc = timed_launch(c, average ? tAverage : tFused, [&] {
        return average ? launch_average(sync_params(c), (int64_t)c->tiles.size(), c->hp.avg_momentum != 0, c->vec,
                                        c->average_nt, c->average_cap, c->stream)
                       : launch_span_of(c, w, c->sync_nt, c->stream);
    });
    if (rc) return rc;
    const ReduceParams r = reduce_params(c, w, c->d_slots, 0, kRing, false);
    rc = timed_launch(c, tSegsum, [&] { return launch_reduce(r, c->stream); });
    if (rc) return rc;
    HIP_TRY(hipEventRecord(c->ring_ev[0], c->stream));
    return ok();
}

// A span, then the reduction of its measurements (if any) into the record slots
// from `slot0` on, then the event of the last of them.  *seq: the timed sequence
// number of the span.
int enqueue_span(adpsgd_ctx *c, const SpanWhen &w, int slot0, bool control, int64_t *seq) {
    int rc = timed_launch(c, -1, [&] { return launch_span_of(c, w, c->sync_nt, c->stream); }, seq, w.n);
    if (rc || measurements(w) == 0) return rc;
    const ReduceParams r = reduce_params(c, w, c->d_slots, slot0, kRing, control);
    rc = timed_launch(c, tSegsum, [&] { return launch_reduce(r, c->stream); }, nullptr, r.n_slots);
    if (rc) return rc;
    HIP_TRY(hipEventRecord(c->ring_ev[(slot0 + r.n_slots - 1) % kRing], c->stream));
    return ok();
}

// Capture the spans of a schedule that no decision moves as a graph: the spans, and
// after each the reduction into as many of the graph's record slots.  No events:
// records are read after the whole graph has run.
int capture_run(adpsgd_ctx *c, const std::vector<SpanWhen> &spans, int64_t n_sync) {
    drop_graph(c);
    if (n_sync > c->gslot_cap) {
        if (c->h_gslots) (void)hipHostFree(c->h_gslots);
        c->h_gslots = c->d_gslots = nullptr;
        c->gslot_cap = 0;
        HIP_TRY(hipHostMalloc((void **)&c->h_gslots, (size_t)n_sync * c->slot_bytes,
                              hipHostMallocMapped | hipHostMallocCoherent));
        HIP_TRY(hipHostGetDevicePointer((void **)&c->d_gslots, c->h_gslots, 0));
        c->gslot_cap = n_sync;
    }
    if (!c->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    const hipStream_t cs = c->cap_stream;
    HIP_TRY(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    hipError_t e = hipSuccess;
    int slot = 0;
    for (const SpanWhen &w : spans) {
        const int m = measurements(w);
        if (m == 0 && !w.merged) {
            e = launch_local_step(step_params(c, w.t, w.n), c->vec, c->nontemporal, c->step_shape, cs);
        } else {
            e = launch_span_of(c, w, c->sync_nt, cs);
            if (e == hipSuccess && m > 0)
                e = launch_reduce(reduce_params(c, w, c->d_gslots, slot, (int)std::max<int64_t>(n_sync, 1), false), cs);
        }
        slot += m;
        if (e != hipSuccess) break;
    }
    hipGraph_t g = nullptr;
    const hipError_t e_end = hipStreamEndCapture(cs, &g);
    if (e == hipSuccess) e = e_end;
    if (e == hipSuccess) e = hipGraphInstantiate(&c->graph_exec, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        c->graph_exec = nullptr;
        return hip_fail(e, "capture the run as a HIP graph");
    }
    c->graph = g;
    return ok();
}

double sum_var(const double *v, int32_t T) {
    double s = 0.0;
    for (int32_t i = 0; i < T; ++i) s += v[i];
    return s;
}

// Contexts created by adpsgd_init and not yet destroyed: a call with any other
// pointer (a destroyed context, say) is refused instead of touching freed memory.
std::mutex g_live_mu;
std::unordered_set<const adpsgd_ctx *> g_live;

int check_ctx(const adpsgd_ctx *c) {
    if (!c) return fail(ADPSGD_EINVAL, "context is NULL");
    std::lock_guard<std::mutex> lock(g_live_mu);
    if (!g_live.count(c)) return fail(ADPSGD_EINVAL, "not a live context (destroyed, or not made by adpsgd_init)");
    return ok();
}

// The context's device made current for the duration of a call, and the
// caller's restored afterwards (a context's buffers, stream and events belong
// to the device that was current at adpsgd_init).
struct DeviceScope {
    int prev = -1;
    explicit DeviceScope(const adpsgd_ctx *c) {
        int cur = -1;
        if (hipGetDevice(&cur) == hipSuccess && cur != c->device && hipSetDevice(c->device) == hipSuccess) prev = cur;
    }
    ~DeviceScope() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
    DeviceScope(const DeviceScope &) = delete;
    DeviceScope &operator=(const DeviceScope &) = delete;
};

// A roctx range for the duration of a call (visible with rocprofv3 --marker-trace).
struct Range {
    explicit Range(const char *name) { roctxRangePushA(name); }
    ~Range() { roctxRangePop(); }
    Range(const Range &) = delete;
    Range &operator=(const Range &) = delete;
};

// Zero the K rows of x and m (P elements each, row_stride apart; the padding
// between rows is the caller's and is left alone), with a fill kernel.
hipError_t zero_rows(const adpsgd_ctx *c) {
    hipError_t e = launch_zero_rows(c->buf.x, c->ld, c->P, c->K, c->vec, c->stream);
    if (e == hipSuccess) e = launch_zero_rows(c->buf.m, c->ld, c->P, c->K, c->vec, c->stream);
    return e;
}

// The fastest of n launch variants on the context's stream: one warm-up launch
// each, then five rounds; a round queues every variant back to back with an
// event between consecutive launches, so each interval is the GPU's time for
// one launch (no host round trip inside it).  The fastest minimum wins.
constexpr int kMaxVariants = 8;

template <class Launch>
hipError_t fastest_variant(adpsgd_ctx *c, int n, Launch launch, int *win) {
    if (n < 1 || n > kMaxVariants) return hipErrorInvalidValue;
    hipEvent_t ev[kMaxVariants + 1] = {};
    hipError_t e = hipSuccess;
    for (int j = 0; j <= n && e == hipSuccess; ++j) e = hipEventCreate(&ev[j]);
    float best[kMaxVariants];
    for (int j = 0; j < n; ++j) best[j] = 3.4e38f;
    for (int j = 0; j < n && e == hipSuccess; ++j) e = launch(j);
    for (int round = 0; round < 5 && e == hipSuccess; ++round) {
        e = hipEventRecord(ev[0], c->stream);
        for (int j = 0; j < n && e == hipSuccess; ++j)
            if ((e = launch(j)) == hipSuccess) e = hipEventRecord(ev[j + 1], c->stream);
        if (e == hipSuccess) e = hipEventSynchronize(ev[n]);
        for (int j = 0; j < n && e == hipSuccess; ++j) {
            float ms = 0.f;
            if ((e = hipEventElapsedTime(&ms, ev[j], ev[j + 1])) == hipSuccess) best[j] = std::min(best[j], ms);
        }
    }
    if (e == hipSuccess) {
        *win = 0;
        for (int j = 1; j < n; ++j)
            if (best[j] < best[*win]) *win = j;
    }
    for (int j = 0; j <= n; ++j)
        if (ev[j]) (void)hipEventDestroy(ev[j]);
    return e;
}

// Time the local step in every launch shape on the context's own buffers (the
// launches step x and m, which the caller zeroes afterwards).
hipError_t tune_step_shape(adpsgd_ctx *c) {
    const StepParams p = step_params(c, 0);
    constexpr int n = (int)(sizeof(kStepShapes) / sizeof(kStepShapes[0]));
    static_assert(n <= kMaxVariants, "more step shapes than the timing helper takes");
    int win = 0;
    const hipError_t e = fastest_variant(
        c, n, [&](int j) { return launch_local_step(p, c->vec, c->nontemporal, kStepShapes[j], c->stream); }, &win);
    if (e == hipSuccess) c->tuned_shape = c->step_shape = kStepShapes[win];
    return e;
}

// The fastest of n launch sequences, each timed in a block of its own: one
// untimed call (which also pays for what the sequence before it left in the
// caches), then `reps` timed calls back to back; two passes over the
// variants, the smaller mean of the two counts.
template <class Launch>
hipError_t fastest_in_blocks(adpsgd_ctx *c, int n, int reps, Launch launch, int *win) {
    if (n < 1 || n > kMaxVariants || reps < 1) return hipErrorInvalidValue;
    hipEvent_t ev[2] = {};
    hipError_t e = hipEventCreate(&ev[0]);
    if (e == hipSuccess) e = hipEventCreate(&ev[1]);
    float best[kMaxVariants];
    for (int j = 0; j < n; ++j) best[j] = 3.4e38f;
    for (int pass = 0; pass < 2 && e == hipSuccess; ++pass)
        for (int j = 0; j < n && e == hipSuccess; ++j) {
            e = launch(j);
            if (e == hipSuccess) e = hipEventRecord(ev[0], c->stream);
            for (int r = 0; r < reps && e == hipSuccess; ++r) e = launch(j);
            if (e == hipSuccess) e = hipEventRecord(ev[1], c->stream);
            if (e == hipSuccess) e = hipEventSynchronize(ev[1]);
            float ms = 0.f;
            if (e == hipSuccess && (e = hipEventElapsedTime(&ms, ev[0], ev[1])) == hipSuccess)
                best[j] = std::min(best[j], ms);
        }
    if (e == hipSuccess) {
        *win = 0;
        for (int j = 1; j < n; ++j)
            if (best[j] < best[*win]) *win = j;
    }
    for (hipEvent_t x : ev)
        if (x) (void)hipEventDestroy(x);
    return e;
}

// Whether spans keep non-temporal accesses.  Beyond 1 GiB of x and m they do
// (measured 6% faster at K = 8, P = 138M).  Between the last-level cache's 256 MB
// and 1 GiB it depends on the problem (four steps with a sync measured 17% faster
// without them at K = 32, P = 1.2M, and 14% slower at K = 8, P = 11.2M), so time
// such spans both ways.  The launches step x and m, which the caller zeroes
// afterwards.
constexpr double kSyncNtTuneMaxBytes = 1024.0 * 1024 * 1024;

hipError_t tune_sync_nt(adpsgd_ctx *c) {
    c->sync_nt = c->nontemporal;
    if (!c->nontemporal || c->tiles.empty() || (double)c->K * (double)c->P * 8.0 > kSyncNtTuneMaxBytes)
        return hipSuccess;
    int win = 0;
    const hipError_t e = fastest_in_blocks(
        c, 2, 6, [&](int j) { return launch_span_of(c, planned(0, 4, 8, false), j == 0, c->stream); }, &win);
    if (e == hipSuccess) c->sync_nt = win == 0;
    return e;
}

// Time the separate sync (mean, broadcast and variance of every tile, no step)
// without and with an LDS cap that holds a CU to kAverageCapWaves resident
// waves and, on x and m of 256 MB to 1 GiB (beyond the last-level cache, see
// tune_sync_nt), with and without non-temporal accesses, on the context's own
// buffers (zeroed again afterwards).
hipError_t tune_average(adpsgd_ctx *c) {
    const int waves = average_tile_waves(c->K);
    if (waves <= 0 || c->tiles.empty()) return hipSuccess;
    const int caps[2] = {0, std::max(1, kAverageCapWaves / waves)};
    const bool both = c->nontemporal && (double)c->K * (double)c->P * 8.0 <= kSyncNtTuneMaxBytes;
    const int n = both ? 4 : 2;   // j: cap caps[j & 1], non-temporal while j < 2 (if at all)
    const SyncParams sp = sync_params(c);
    const int64_t n_tiles = (int64_t)c->tiles.size();
    int win = 0;
    const hipError_t e = fastest_in_blocks(
        c, n, 3,
        [&](int j) {
            return launch_average(sp, n_tiles, c->hp.avg_momentum != 0, c->vec, c->nontemporal && j < 2, caps[j & 1],
                                  c->stream);
        },
        &win);
    if (e == hipSuccess) {
        c->average_cap = caps[win & 1];
        c->average_nt = c->nontemporal && win < 2;
    }
    return e;
}

}  // namespace

extern "C" const char *adpsgd_last_error(void) { return g_last_error.c_str(); }

extern "C" int64_t adpsgd_padded_row_stride(int64_t P) {
    if (P <= 0) return 0;
    const int64_t n = (P - 1) / 256 + 1;
    return 256 * (n | 1);
}

extern "C" size_t adpsgd_workspace_bytes(int32_t K, int64_t P, int32_t T, const int64_t *offsets) {
    std::string why;
    if (!shape_valid(K, P, T, offsets, &why)) return 0;
    return layout_for(count_plan(T, offsets), T).total;
}

extern "C" int adpsgd_init(int32_t K, int64_t P, const int64_t *offsets, int32_t T, const adpsgd_hparams *hp,
                           const adpsgd_buffers *buf, adpsgd_ctx **out) {
    Range range_("adpsgd_init");
    std::string why;
    if (!out) return fail(ADPSGD_EINVAL, "out is NULL");
    *out = nullptr;
    if (!shape_valid(K, P, T, offsets, &why)) return fail(ADPSGD_EINVAL, why);
    if (!hparams_valid(hp, &why)) return fail(ADPSGD_EINVAL, why);
    if (!buf) return fail(ADPSGD_EINVAL, "buffers is NULL");
    if (P > 0 && (!buf->x || !buf->m || !buf->h || !buf->xstar))
        return fail(ADPSGD_EINVAL, "x, m, h and xstar must be non-NULL");
    if (!aligned(buf->x, 16) || !aligned(buf->m, 16) || !aligned(buf->h, 16) || !aligned(buf->xstar, 16))
        return fail(ADPSGD_EINVAL, "x, m, h and xstar must be 16-byte aligned");
    if (buf->row_stride < 0 || (buf->row_stride > 0 && buf->row_stride < P))
        return fail(ADPSGD_EINVAL, "row_stride must be 0 or >= P");
    const Plan plan = count_plan(T, offsets);
    // tile indices are 32-bit in the chunk table (P / 4 < 2^32 keeps them far below)
    if (plan.n_tiles >= (int64_t(1) << 31)) return fail(ADPSGD_EINVAL, "too many sync tiles");
    const Layout lay = layout_for(plan, T);
    if (!buf->workspace || !aligned(buf->workspace, 256)) return fail(ADPSGD_EINVAL, "workspace must be 256-byte aligned");
    if (buf->workspace_bytes < lay.total)
        return fail(ADPSGD_EINVAL, "workspace too small: need " + std::to_string(lay.total) + " bytes");

    adpsgd_ctx *c = new (std::nothrow) adpsgd_ctx();
    if (!c) return fail(ADPSGD_EINVAL, "out of host memory");
    c->K = K;
    c->P = P;
    c->T = T;
    c->offsets.assign(offsets, offsets + T + 1);
    build_plan(T, offsets, plan.chunk_tiles, &c->tiles, &c->chunks, &c->chunk_begin);
    c->chunks_are_tiles = plan.chunk_tiles == 1;
    c->hp = *hp;
    c->buf = *buf;
    c->stream = (hipStream_t)buf->stream;
    c->ld = buf->row_stride > 0 ? buf->row_stride : P;
    c->vec = (c->ld % 4) == 0;
    // x and m beyond the 256 MB last-level cache: stream them past the caches
    c->nontemporal = (double)K * (double)P * 8.0 > 256.0 * 1024 * 1024;
    c->sync_nt = c->average_nt = c->nontemporal;   // until timed
    c->rk = round_keys(hp->seed);
    char *ws = (char *)buf->workspace;
    c->d_tiles = (Tile *)(ws + lay.tiles);
    c->d_chunks = (Chunk *)(ws + lay.chunks);
    c->d_chunk_begin = (int32_t *)(ws + lay.chunk_begin);
    c->d_large = (int32_t *)(ws + lay.large);
    c->d_win_begin = (int32_t *)(ws + lay.win_begin);
    c->d_win_partials = (double *)(ws + lay.win_partials);
    if (reduce_windows(T, c->chunk_begin.data(), &c->win_begin) != plan.n_windows) {
        release(c);
        return fail(ADPSGD_EINVAL, "internal: window table disagrees with the workspace plan");
    }
    for (int32_t tau = 0; tau < T; ++tau)
        if (c->chunk_begin[tau + 1] - c->chunk_begin[tau] > kSmallTensorChunks) c->large.push_back(tau);
    c->d_tile_partials = (double *)(ws + lay.tile_partials);
    c->d_chunk_partials = (double *)(ws + lay.chunk_partials);
    c->d_acc = (double *)(ws + lay.acc);
    c->d_sums = (double *)(ws + lay.sums);
    c->n_slots = plan.n_slots;
    c->d_sched = (SchedState *)(ws + lay.sched);
    c->d_chunk_seg = (int32_t *)(ws + lay.chunk_seg);
    if (!chunk_segments(c->tiles, plan.n_aligned, &c->chunk_seg)) {
        release(c);
        return fail(ADPSGD_EINVAL, "internal: the tile table does not cover every aligned chunk");
    }
    c->slot_bytes = slot_bytes_for(T);

    auto bail = [&](hipError_t e, const char *what) {
        int rc = hip_fail(e, what);
        std::string msg = g_last_error;
        release(c);
        g_last_error = msg;
        return rc;
    };
    hipError_t e;
    if ((e = hipGetDevice(&c->device)) != hipSuccess) return bail(e, "hipGetDevice");
    // the reduction writes its records straight into coherent pinned memory
    if ((e = hipHostMalloc((void **)&c->h_slots, (size_t)kRing * c->slot_bytes,
                           hipHostMallocMapped | hipHostMallocCoherent)) != hipSuccess)
        return bail(e, "hipHostMalloc");
    if ((e = hipHostGetDevicePointer((void **)&c->d_slots, c->h_slots, 0)) != hipSuccess)
        return bail(e, "hipHostGetDevicePointer");
    if ((e = hipHostMalloc((void **)&c->h_sched, sizeof(SchedState), hipHostMallocDefault)) != hipSuccess)
        return bail(e, "hipHostMalloc");
    for (auto &ev : c->ring_ev)
        if ((e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess) return bail(e, "hipEventCreate");
    if (!c->tiles.empty() &&
        (e = hipMemcpyAsync(c->d_tiles, c->tiles.data(), sizeof(Tile) * c->tiles.size(), hipMemcpyHostToDevice,
                            c->stream)) != hipSuccess)
        return bail(e, "copy tile table");
    if (!c->chunks.empty() &&
        (e = hipMemcpyAsync(c->d_chunks, c->chunks.data(), sizeof(Chunk) * c->chunks.size(), hipMemcpyHostToDevice,
                            c->stream)) != hipSuccess)
        return bail(e, "copy chunk table");
    if ((e = hipMemcpyAsync(c->d_chunk_begin, c->chunk_begin.data(), sizeof(int32_t) * (T + 1),
                            hipMemcpyHostToDevice, c->stream)) != hipSuccess)
        return bail(e, "copy chunk offsets");
    if ((e = hipMemcpyAsync(c->d_chunk_seg, c->chunk_seg.data(), sizeof(int32_t) * c->chunk_seg.size(),
                            hipMemcpyHostToDevice, c->stream)) != hipSuccess)
        return bail(e, "copy the aligned chunks' tiles");
    if (!c->large.empty() &&
        (e = hipMemcpyAsync(c->d_large, c->large.data(), sizeof(int32_t) * c->large.size(), hipMemcpyHostToDevice,
                            c->stream)) != hipSuccess)
        return bail(e, "copy large-tensor list");
    if (!c->win_begin.empty() &&
        (e = hipMemcpyAsync(c->d_win_begin, c->win_begin.data(), sizeof(int32_t) * c->win_begin.size(),
                            hipMemcpyHostToDevice, c->stream)) != hipSuccess)
        return bail(e, "copy window table");
    if (P > 0) {
        if ((e = launch_init_problem(buf->h, buf->xstar, P, hp->seed, hp->h_lo, hp->h_hi, c->stream)) != hipSuccess)
            return bail(e, "init_problem launch");
        if ((e = zero_rows(c)) != hipSuccess) return bail(e, "zero x and m");
        if ((double)K * (double)P >= kTuneMinElems) {
            if ((e = tune_step_shape(c)) != hipSuccess) return bail(e, "time the local step");
            if ((e = tune_sync_nt(c)) != hipSuccess) return bail(e, "time the fused step + sync");
            if ((e = tune_average(c)) != hipSuccess) return bail(e, "time the separate sync");
            if ((e = zero_rows(c)) != hipSuccess) return bail(e, "zero x and m");
        }
    }
    if ((e = hipStreamSynchronize(c->stream)) != hipSuccess) return bail(e, "hipStreamSynchronize");
    c->st = adpsgd_state{};
    c->st.p = hp->p_init;
    {
        std::lock_guard<std::mutex> lock(g_live_mu);
        g_live.insert(c);
    }
    *out = c;
    return ok();
}

extern "C" int adpsgd_reset(adpsgd_ctx *c) {
    if (int rc = check_ctx(c)) return rc;
    DeviceScope dev_(c);
    HIP_TRY(zero_rows(c));
    c->st = adpsgd_state{};
    c->st.p = c->hp.p_init;
    return ok();
}

extern "C" int adpsgd_local_steps(adpsgd_ctx *c, int32_t n) {
    Range range_("adpsgd_local_steps");
    if (int rc = check_ctx(c)) return rc;
    DeviceScope dev_(c);
    if (n < 0) return fail(ADPSGD_EINVAL, "n must be >= 0");
    if (c->st.t + n > kMaxCounter) return fail(ADPSGD_EINVAL, "step index would reach 2^32");
    if (int rc = enqueue_steps(c, c->st.t, n)) return rc;
    c->st.t += n;
    c->st.cnt += n;
    // a constant period that switches at p_switch_step does so for the state too
    if (n > 0) c->st.p = period_at(rule_of(&c->hp), c->st.p, c->st.t - 1);
    return ok();
}

static int sync_now(adpsgd_ctx *c, bool fused, double *var_out) {
    Range range_("adpsgd_sync");
    if (int rc = check_ctx(c)) return rc;
    DeviceScope dev_(c);
    if (!var_out) return fail(ADPSGD_EINVAL, "var_out is NULL");
    if (fused && c->st.t + 1 > kMaxCounter) return fail(ADPSGD_EINVAL, "step index would reach 2^32");
    if (int rc = enqueue_sync(c, !fused, c->st.t)) return rc;
    HIP_TRY(hipEventSynchronize(c->ring_ev[0]));
    std::memcpy(var_out, slot_host(c, 0) + kSlotHdrBytes, sizeof(double) * c->T);
    if (fused) {
        c->st.p = period_at(rule_of(&c->hp), c->st.p, c->st.t);
        c->st.t += 1;
    }
    c->st.cnt = 0;
    return ok();
}

extern "C" int adpsgd_average(adpsgd_ctx *c, double *var_out) { return sync_now(c, false, var_out); }

extern "C" int adpsgd_step_average(adpsgd_ctx *c, double *var_out) { return sync_now(c, true, var_out); }

extern "C" int adpsgd_schedule(adpsgd_ctx *c, const double *var, int32_t *next_period) {
    if (int rc = check_ctx(c)) return rc;
    if (!var) return fail(ADPSGD_EINVAL, "var is NULL");
    if (c->st.t < 1) return fail(ADPSGD_ESTATE, "no step has been taken yet");
    int rc = adpsgd_sched_on_sync(&c->hp, &c->st, c->st.t - 1, sum_var(var, c->T), nullptr);
    if (next_period) *next_period = c->st.p;
    return rc;
}

// Algorithm 2 for n_steps steps (adpsgd_run, adpsgd_run_traced).
//
// The host plans launches from its replay of the schedule.  While that is exact
// a launch takes as many steps and syncs as it can (plan_span), up to and with
// the first sync whose outcome may move p.  What follows such a sync is a span
// that the device ends: it takes steps until Algorithm 2's counter (read from the
// device copy of the controller state) says that a sync is due, so neither its
// length nor, for the launch after it, its first step need be known to the host.
// The reduction behind every span sums the variances and takes Algorithm 2's
// decisions on the device, so the GPU never waits for a host round trip.  Every
// record is read back in order, replayed by the host controller (same rules,
// same fp64 operations) and checked against the device's decision.  A traced run
// measures every step of its launches.
static int run_impl(adpsgd_ctx *c, int64_t n_steps, adpsgd_sync_rec *log, int64_t log_cap, double *var_log,
                    adpsgd_step_rec *trace, int64_t trace_cap, int64_t *n_syncs) {
    Range range_("adpsgd_run");
    if (int rc = check_ctx(c)) return rc;
    DeviceScope dev_(c);
    if (n_steps < 0 || log_cap < 0 || trace_cap < 0) return fail(ADPSGD_EINVAL, "n_steps and capacities must be >= 0");
    if (log_cap > 0 && !log) return fail(ADPSGD_EINVAL, "log is NULL with log_cap > 0");
    if (trace_cap > 0 && !trace) return fail(ADPSGD_EINVAL, "trace is NULL with trace_cap > 0");
    if (c->st.t + n_steps > kMaxCounter) return fail(ADPSGD_EINVAL, "step index would reach 2^32");

    const adpsgd_hparams &hp = c->hp;
    const SchedRule rule = rule_of(&hp);
    const bool traced = trace != nullptr;
    const bool adaptive = hp.period_mode == ADPSGD_PERIOD_ADAPTIVE;
    const bool by_step = c->policy == ADPSGD_LAUNCH_DEVICE;   // every step decided on the device
    const bool control = adaptive || by_step;   // the controller state lives on the device
    const bool merge = !by_step && c->K > 1 && span_in_registers(c->K);
    const int64_t t0 = c->st.t, end = t0 + n_steps;
    const Planner planner{rule, end, c->n_slots, traced, by_step, c->policy == ADPSGD_LAUNCH_HOST,
                          span_in_registers(c->K), merge};

    // A run whose schedule is fixed in advance (constant-period modes) on a
    // small, launch-bound problem replays a captured graph of the whole run.
    const bool graph_mode = c->policy == ADPSGD_LAUNCH_HYBRID && !traced && !c->timing && n_steps > 0 &&
                            n_steps <= kGraphMaxSteps && !adaptive && (double)c->K * (double)c->P < kGraphMaxElems;

    // A launch in flight: what it takes, and its record slots (slot0 < 0: none).
    struct Entry { SpanWhen w; int slot0, n_slots; int64_t seq; };
    std::deque<Entry> inflight;
    adpsgd_state known = c->st;   // the host controller after every accounted step
    int64_t n_done = 0, n_launches = 0, next_slot = 0, slots_used = 0;
    bool dirty = false;           // a record was read: the launches ahead are known better
    int status = ADPSGD_OK;

    auto slot_rec = [&](int slot) -> const char * {
        return graph_mode ? c->h_gslots + (size_t)slot * c->slot_bytes : slot_host(c, slot % kRing);
    };
    // Account for one measurement: step t, in record slot `slot`.
    auto account_slot = [&](int slot, int64_t t, bool due) -> int {
        SlotHdr hdr;
        std::memcpy(&hdr, slot_rec(slot), sizeof hdr);
        const double *var = reinterpret_cast<const double *>(slot_rec(slot) + kSlotHdrBytes);
        if (hdr.t != t || (hdr.due != 0) != due)
            return fail(ADPSGD_ESTATE, "device and host schedules disagree at step " + std::to_string(t));
        const double gamma = adpsgd_lr(&hp, t);
        if (traced && t - t0 < trace_cap)
            trace[t - t0] = adpsgd_step_rec{t, due ? 1 : 0, known.p, hdr.S, hdr.GN, gamma};
        if (!due) return ADPSGD_OK;
        const int32_t p_in_force = known.p;
        double margin = std::numeric_limits<double>::quiet_NaN();
        const int rc = adpsgd_sched_on_sync(&hp, &known, t, hdr.S, &margin);
        if (n_done < log_cap) {
            log[n_done] = adpsgd_sync_rec{t, p_in_force, 0, hdr.S, known.C2, gamma, margin};
            if (var_log) std::memcpy(var_log + (size_t)n_done * c->T, var, sizeof(double) * c->T);
        }
        ++n_done;
        // (a non-finite S still restarted the counter; only p and C2 stay)
        if (rc) return hdr.status == rc ? rc : fail(ADPSGD_ESTATE, "device and host disagree on a non-finite S");
        if (hdr.status != ADPSGD_OK ||
            (control && (hdr.p_next != known.p || hdr.C2 != known.C2 || hdr.nC2 != known.nC2)))
            return fail(ADPSGD_ESTATE, "device and host controllers disagree at step " + std::to_string(t));
        return ADPSGD_OK;
    };
    // Account for a finished launch: replay its steps on the host and check the
    // device's records against the replay.  After a failure the remaining records
    // are still accounted for (the steps ran); the first error is the one reported.
    auto account = [&](const Entry &e) -> int {
        int first = ADPSGD_OK;
        int32_t n = e.w.n, n_sync = 0;
        if (e.w.device) {
            SlotHdr hdr;
            std::memcpy(&hdr, slot_rec(e.slot0), sizeof hdr);
            n = hdr.n;
            if (n < 0 || n > e.w.n || known.t + n > end) return fail(ADPSGD_ESTATE, "internal: a launch's record is not whole");
        }
        int slot = e.slot0;
        for (int32_t j = 0; j < n; ++j) {
            const int64_t t = known.t;
            int32_t due = 0;
            (void)adpsgd_sched_step(&hp, &known, &due);
            // a launch that the device ends, ends with its sync and not before
            // (or at the most steps it was given)
            const bool planned_due = e.w.device ? j == n - 1 && due : (e.w.syncs >> j) & 1;
            const bool cut = e.w.device && j == n - 1 && !due && n < e.w.n && known.t < end && e.w.known;
            if ((due != 0) != planned_due || cut) {
                if (!first) first = fail(ADPSGD_ESTATE, "device and host schedules disagree at step " + std::to_string(t));
                if (due) known.cnt = 0;
                continue;
            }
            n_sync += due;
            if (!due && !e.w.measure) continue;
            const int rc = account_slot(slot++, t, due != 0);
            if (rc && !first) first = rc;
        }
        set_span(c, e.seq, e.w.n, traced ? tTrace : tStep, n, n_sync);
        return first;
    };

    if (graph_mode) {
        // the launches, from the host controller alone (no decision moves p)
        std::vector<SpanWhen> spans;
        adpsgd_state pl = known;
        int64_t n_sync = 0;
        while (pl.t < end) {
            spans.push_back(planner.span(&pl, merge && !spans.empty() && pl.cnt == 0));
            n_sync += measurements(spans.back());
        }
        const int64_t key[7] = {t0, n_steps, known.cnt, known.p, c->step_shape.block, c->step_shape.lds,
                                c->step_shape.row_chunks};
        if (!c->graph_exec || std::memcmp(key, c->graph_key, sizeof key) != 0) {
            Range cap_("adpsgd_run: capture a graph");
            if (int rc = capture_run(c, spans, n_sync)) return rc;
            std::memcpy(c->graph_key, key, sizeof key);
            ++c->graph_captures;
        }
        ++c->graph_replays;
        {
            Range replay_("adpsgd_run: graph replay");
            HIP_TRY(hipGraphLaunch(c->graph_exec, c->stream));
            HIP_TRY(hipStreamSynchronize(c->stream));
        }
        int slot = 0;
        for (const SpanWhen &w : spans) {
            const int rc = account(Entry{w, slot, measurements(w), -1});
            if (rc && status == ADPSGD_OK) status = rc;
            slot += measurements(w);
        }
        c->st = known;
        if (n_syncs) *n_syncs = n_done;
        return status != ADPSGD_OK ? status : ok();
    }

    if (n_steps > 0 && control) {
        *c->h_sched = SchedState{known.t, known.cnt, known.nC2, known.C2, known.p, 0};
        HIP_TRY(hipMemcpyAsync(c->d_sched, c->h_sched, sizeof(SchedState), hipMemcpyHostToDevice, c->stream));
    }

    // Account for every launch at the front that is finished (with `wait`, for
    // at least the first one that has records).
    auto drain = [&](bool wait) -> int {
        while (!inflight.empty()) {
            const Entry e = inflight.front();
            if (e.slot0 >= 0) {
                const hipEvent_t ev = c->ring_ev[(e.slot0 + e.n_slots - 1) % kRing];
                hipError_t q;
                if (wait) {
                    Range wait_("adpsgd_run: wait for a record");
                    q = hipEventSynchronize(ev);
                } else {
                    q = hipEventQuery(ev);
                }
                if (q == hipErrorNotReady) break;
                if (q != hipSuccess) return hip_fail(q, "wait for a record");
                wait = false;
                slots_used -= e.n_slots;
                dirty = true;
            }
            inflight.pop_front();
            const int rc = account(e);
            if (rc && status == ADPSGD_OK) status = rc;
        }
        return ADPSGD_OK;
    };

    Planner::Ahead ahead = Planner::known(known);   // after every launch in flight

    int hard = ADPSGD_OK;  // a HIP failure: stop at once
    while (hard == ADPSGD_OK) {
        if (n_launches % kPollEvery == 0) {
            if ((hard = drain(false))) break;
            if (c->timing && (hard = harvest(c, false))) break;
        }
        if (dirty) {
            ahead = Planner::known(known);
            for (const Entry &e : inflight) planner.pass(&ahead, e.w);
            dirty = false;
        }
        if (status != ADPSGD_OK || ahead.t_hi >= end) {
            // (launches the device ends may stop short of the end: then there is more to do)
            if (inflight.empty()) break;
            hard = drain(true);
            continue;
        }

        Entry e{SpanWhen{}, -1, 0, -1};
        bool wait = !planner.next(ahead, n_launches == 0, &e.w);
        if (!wait) {
            e.n_slots = measurements(e.w);
            wait = slots_used + e.n_slots > kRing || (int64_t)inflight.size() >= kMaxInflight;
        }
        if (wait) {
            if (inflight.empty()) { hard = fail(ADPSGD_ESTATE, "internal: nothing in flight to wait for"); break; }
            hard = drain(true);
            continue;
        }
        if (e.n_slots == 0 && !e.w.merged) {
            hard = enqueue_steps(c, e.w.t, e.w.n);
        } else if (e.n_slots == 0) {
            hard = enqueue_span(c, e.w, 0, control, &e.seq);
        } else {
            e.slot0 = (int)(next_slot % kRing);
            next_slot += e.n_slots;
            slots_used += e.n_slots;
            hard = enqueue_span(c, e.w, e.slot0, control, &e.seq);
        }
        if (hard) break;
        inflight.push_back(e);
        planner.pass(&ahead, e.w);
        ++n_launches;
    }
    // whatever was enqueued runs to completion and is accounted for
    hipError_t e = hipStreamSynchronize(c->stream);
    while (e == hipSuccess && hard == ADPSGD_OK && !inflight.empty()) hard = drain(true);
    if (e == hipSuccess && hard == ADPSGD_OK && merge && n_launches > 0 && known.t < end && known.cnt == 0) {
        // stopped by a non-finite S behind a sync: whole rows again
        e = launch_spread_row(c->buf.x, c->ld, c->P, c->K, c->vec, c->stream);
        if (e == hipSuccess && hp.avg_momentum)
            e = launch_spread_row(c->buf.m, c->ld, c->P, c->K, c->vec, c->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    }
    c->st = known;
    if (n_syncs) *n_syncs = n_done;
    if (hard != ADPSGD_OK) return hard;
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    if (status != ADPSGD_OK) return status;
    return ok();
}

extern "C" int adpsgd_run(adpsgd_ctx *c, int64_t n_steps, adpsgd_sync_rec *log, int64_t log_cap, double *var_log,
                          int64_t *n_syncs) {
    return run_impl(c, n_steps, log, log_cap, var_log, nullptr, 0, n_syncs);
}

extern "C" int adpsgd_run_traced(adpsgd_ctx *c, int64_t n_steps, adpsgd_sync_rec *log, int64_t log_cap,
                                 double *var_log, adpsgd_step_rec *trace, int64_t trace_cap, int64_t *n_syncs) {
    if (!trace) return fail(ADPSGD_EINVAL, "trace is NULL");
    return run_impl(c, n_steps, log, log_cap, var_log, trace, trace_cap, n_syncs);
}

extern "C" int adpsgd_get_state(const adpsgd_ctx *c, adpsgd_state *out) {
    if (int rc = check_ctx(c)) return rc;
    if (!out) return fail(ADPSGD_EINVAL, "out is NULL");
    *out = c->st;
    return ok();
}

extern "C" int adpsgd_set_state(adpsgd_ctx *c, const adpsgd_state *in) {
    if (int rc = check_ctx(c)) return rc;
    if (!in) return fail(ADPSGD_EINVAL, "state is NULL");
    if (in->t < 0 || in->t >= kMaxCounter || in->cnt < 0 || in->nC2 < 0 || in->p < 1 || in->p > p_max_of(&c->hp) ||
        !std::isfinite(in->C2))
        return fail(ADPSGD_EINVAL, "invalid state");
    c->st = *in;
    return ok();
}

extern "C" int adpsgd_set_step_launch(adpsgd_ctx *c, int32_t block, int32_t lds_bytes, int32_t row_chunks) {
    if (int rc = check_ctx(c)) return rc;
    if (block == 0) {
        c->step_shape = c->tuned_shape;
        return ok();
    }
    bool known = false;
    for (int b : kStepBlocks) known = known || b == block;
    if (!known) return fail(ADPSGD_EINVAL, "block must be 0, 64, 128 or 256");
    if (lds_bytes < 0 || lds_bytes > kMaxStepLds) return fail(ADPSGD_EINVAL, "lds_bytes must be in [0, 65536]");
    if (row_chunks < 1 || row_chunks > kMaxRowChunks) return fail(ADPSGD_EINVAL, "row_chunks must be in [1, 4096]");
    c->step_shape = StepShape{block, lds_bytes, row_chunks};
    return ok();   // (a captured run keys on the shape, so it is captured again)
}

extern "C" int adpsgd_get_step_launch(const adpsgd_ctx *c, int32_t *block, int32_t *lds_bytes,
                                      int32_t *row_chunks) {
    if (int rc = check_ctx(c)) return rc;
    if (!block || !lds_bytes || !row_chunks) return fail(ADPSGD_EINVAL, "block, lds_bytes or row_chunks is NULL");
    *block = c->step_shape.block;
    *lds_bytes = c->step_shape.lds;
    *row_chunks = c->step_shape.row_chunks;
    return ok();
}

extern "C" int adpsgd_set_launch_policy(adpsgd_ctx *c, int32_t policy) {
    if (int rc = check_ctx(c)) return rc;
    if (policy != ADPSGD_LAUNCH_HYBRID && policy != ADPSGD_LAUNCH_DEVICE && policy != ADPSGD_LAUNCH_HOST)
        return fail(ADPSGD_EINVAL, "unknown launch policy");
    c->policy = policy;
    return ok();
}

extern "C" int adpsgd_set_timing(adpsgd_ctx *c, int32_t every) {
    if (int rc = check_ctx(c)) return rc;
    DeviceScope dev_(c);
    if (every < 0) return fail(ADPSGD_EINVAL, "every must be >= 0");
    HIP_TRY(hipStreamSynchronize(c->stream));
    if (int rc = harvest(c, true)) return rc;
    c->timing = every != 0;
    c->timing_every = every > 0 ? every : 1;
    for (int i = 0; i < tKinds; ++i) { c->t_ms[i] = 0.0; c->t_n[i] = 0; }
    for (auto &n : c->class_seen) n = 0;
    for (auto &n : c->class_timed) n = 0;
    c->graph_captures = c->graph_replays = 0;
    return ok();
}

extern "C" int adpsgd_get_timing(adpsgd_ctx *c, adpsgd_timing *out) {
    if (int rc = check_ctx(c)) return rc;
    DeviceScope dev_(c);
    if (!out) return fail(ADPSGD_EINVAL, "out is NULL");
    HIP_TRY(hipStreamSynchronize(c->stream));
    if (int rc = harvest(c, true)) return rc;
    *out = adpsgd_timing{c->t_ms[tStep],  c->t_n[tStep],   c->t_ms[tFused],  c->t_n[tFused],
                         c->t_ms[tAverage], c->t_n[tAverage], c->t_ms[tSegsum], c->t_n[tSegsum],
                         c->t_ms[tTrace], c->t_n[tTrace], c->graph_captures, c->graph_replays};
    return ok();
}

extern "C" int adpsgd_destroy(adpsgd_ctx *c) {
    if (!c) return ok();
    {
        std::lock_guard<std::mutex> lock(g_live_mu);
        if (!g_live.erase(c)) return fail(ADPSGD_EINVAL, "not a live context (destroyed twice?)");
    }
    hipError_t e;
    {
        DeviceScope dev_(c);
        e = hipStreamSynchronize(c->stream);
        release(c);
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    return ok();
}

extern "C" int adpsgd_philox_dump(uint64_t seed, uint32_t c1, uint32_t c2, uint32_t c3, int64_t g0, int64_t n_groups,
                                  uint32_t *dev_out, void *stream) {
    if (n_groups < 0 || g0 < 0 || g0 + n_groups > kMaxCounter) return fail(ADPSGD_EINVAL, "bad group range");
    if (n_groups > 0 && (!dev_out || !aligned(dev_out, 16))) return fail(ADPSGD_EINVAL, "dev_out must be 16-byte aligned");
    HIP_TRY(launch_philox_dump(seed, c1, c2, c3, g0, n_groups, dev_out, (hipStream_t)stream));
    return ok();
}

extern "C" int adpsgd_normal_dump(uint64_t seed, uint32_t c1, uint32_t c2, uint32_t c3, int64_t g0, int64_t n_groups,
                                  float *dev_out, void *stream) {
    if (n_groups < 0 || g0 < 0 || g0 + n_groups > kMaxCounter) return fail(ADPSGD_EINVAL, "bad group range");
    if (n_groups > 0 && (!dev_out || !aligned(dev_out, 16))) return fail(ADPSGD_EINVAL, "dev_out must be 16-byte aligned");
    HIP_TRY(launch_normal_dump(seed, c1, c2, c3, g0, n_groups, dev_out, (hipStream_t)stream));
    return ok();
}
