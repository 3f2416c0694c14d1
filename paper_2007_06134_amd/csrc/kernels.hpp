// Launch interface between the host runtime and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "rng.hpp"
#include "schedule.hpp"

namespace adpsgd {

constexpr int kBlock = 256;          // threads per workgroup of the streaming kernels
constexpr int64_t kTileElems = 256;  // sync tiles are cut at multiples of 256 elements,
                                     // so a tile spans at most 64 float4 groups (one wave)
constexpr int32_t kChunkTiles = 1024;  // tiles per first-level chunk of the variance sum
// Chunk partials the final reduction block holds in LDS at once.
constexpr int32_t kFinishWindow = 2048;
// Up to this many tiles (one LDS window), every tile is its own chunk: the tile
// partials are the chunk partials and the first reduction launch is skipped.
// (Above it, the one finishing block reading every tile partial costs more
// than the chunk launch: 22 us against 9 us for the pair at 5080 tiles.)
constexpr int64_t kDirectMaxTiles = kFinishWindow;
constexpr int32_t kSmallTensorChunks = 32;  // larger tensors are summed by a wave, not a thread
// Work-items per launch at most; a grid beyond it is issued in pieces of whole
// 8-block groups, so the blocks keep their XCD order across the pieces.
constexpr int64_t kMaxLaunchItems = int64_t(1) << 31;

// One sync tile: a contiguous element range inside one tensor.
struct Tile {
    int64_t start;
    int32_t len;
    int32_t tensor;
};

// Consecutive tiles of one tensor whose partials are summed together.
struct Chunk {
    int32_t first;
    int32_t count;
    int32_t tensor;
    int32_t pad_;
};

// Everything a local step needs.  Replicas are rows of x and m, ld elements apart.
struct StepParams {
    float *x;
    float *m;
    const float *h;
    const float *xs;
    int64_t ld;        // row stride of x and m in elements (>= P)
    int64_t P;
    int64_t n_groups;  // ceil(P / 4)
    int32_t K;
    uint32_t t;        // first step's index (Philox counter word 2)
    float sigma_r;     // sigma sqrt(2 ln 2) (see add_noise2)
    float mu, wd;
    int32_t n;         // steps of this launch: t .. t + n - 1 (k_local_step; see SpanWhen for k_span)
    RoundKeys rk;
    // Chunks of one worker's row that an XCD takes one after another before
    // the next worker's (the local step's block order; set by
    // launch_local_step, ignored by the sync kernels).
    int32_t row_chunks;
    // First block of this launch: a dispatch counts its grid in 32-bit
    // work-items, so larger grids go out as several launches (the launchers
    // below set it; callers leave it 0).
    int64_t block0;
    float gamma[kSpanSteps];  // the rates of steps t, t + 1, ...
};

// (The rates come last in every kernel's arguments, so that what all of its waves
// read first lies together.)
struct SyncParams {
    const Tile *tiles;
    double *partials;  // [2 n_tiles]: per tile, sum of sum_k (xbar - x_k)^2, gradient norm^2
    // k_span and k_average (not the loop kernel) take one block per aligned
    // chunk of kTileElems elements, [c kTileElems, (c + 1) kTileElems) cut at P,
    // whatever tensors it holds: its tiles are chunk_seg[c] .. chunk_seg[c+1]-1
    // (every chunk holds at least one), so a tensor boundary inside a chunk
    // costs no block of its own.
    const int32_t *chunk_seg;  // [n_chunks + 1]
    int64_t n_chunks;          // ceil(P / kTileElems)
    StepParams s;              // x, m, P, K; the step fields are used by spans
};

struct SpanControl {
    int64_t slot_stride;       // doubles from one measurement's tile partials to the next's
    const SchedState *sched;   // (when.device) the controller state
    SpanWhen when;             // s.t = when.t, s.gamma[0] its rate
    int32_t avg_m;             // 1: a sync also averages the momentum buffers
    int32_t pad_;
    SchedRule rule;
};
struct SpanParams : SpanControl, SyncParams {};

// Launch shapes of the local step: threads per block (= float4 groups per
// block), an LDS reservation per block, and the block order.  The kernel uses
// no LDS; the reservation only holds a CU to floor(160 KB / lds) resident
// blocks, and fewer waves in flight can stream HBM slightly faster.  The
// blocks of a chunk (block groups of every worker's row) go to one XCD;
// row_chunks = S: an XCD takes S chunks of one worker's row, then the same S
// chunks of the next worker's, so that each row is streamed in longer runs.
// The grid size for n_groups groups, K workers and a shape is
// local_step_blocks.
struct StepShape {
    int block;
    int lds;
    int row_chunks;
};
constexpr int kStepBlocks[] = {64, 128, 256};
constexpr int kMaxStepLds = 64 * 1024;
constexpr int kMaxRowChunks = 4096;
// The shapes adpsgd_init times: the three block sizes with one chunk per row
// run, 64-thread blocks held to 20 per CU (8 KB each), and those with runs of
// 16, 32 and 64 chunks.
// A launch of n >= kUncappedSteps steps leaves the LDS reservation out: it is
// bound by arithmetic, not by HBM, and wants every wave it can hold (measured
// with and without the 8 KB reservation, K = 8, P = 138M: 1 step 2.97 and 3.03
// ms, 2 steps 3.01 and 3.05, 3 steps 3.18 and 3.10, 4 steps 3.55 and 3.27).
constexpr int kUncappedSteps = 3;
constexpr StepShape kStepShapes[] = {{64, 0, 1},     {64, 8192, 1},  {128, 0, 1},   {256, 0, 1},
                                     {64, 8192, 16}, {64, 8192, 32}, {64, 8192, 64}};
int64_t local_step_blocks(int64_t n_groups, int32_t K, const StepShape &shape);
// vec: rows are 16-byte aligned (row stride % 4 == 0) so full groups use
// dwordx4; shape: block one of kStepBlocks, lds in [0, kMaxStepLds],
// row_chunks in [1, kMaxRowChunks]; p.n in [1, kSpanSteps] (hipErrorInvalidValue otherwise).
hipError_t launch_local_step(const StepParams &p, bool vec, bool nontemporal, const StepShape &shape,
                             hipStream_t st);
// The synchronization alone.  avg_m: the momentum buffers too.  cap > 0 reserves
// LDS (160 KB per CU on gfx950) so that at most cap blocks are resident per CU;
// 0: none.  The loop kernel (K above 128, and K = 3) ignores nontemporal and cap.
hipError_t launch_average(const SyncParams &p, int64_t n_tiles, bool avg_m, bool vec, bool nontemporal, int cap,
                          hipStream_t st);
// Workers whose replicas k_span and k_average hold in the registers of one block.
constexpr int kMaxRegisterK = 128;
constexpr int kSimds = 1024;   // of the 256 CUs
// The span p.when; vec as for launch_local_step, but whole chunks of unaligned rows move
// with dwordx4 too.  With K above kMaxRegisterK a span that the device ends has
// n = 1; a planned one goes out as plain steps (step_nt, shape as for
// launch_local_step) and one loop kernel per measured step.
bool span_in_registers(int K);
hipError_t launch_span(const SpanParams &p, int64_t n_tiles, bool vec, bool nontemporal, bool step_nt,
                       const StepShape &shape, hipStream_t st);
// chunk_seg (SyncParams) of a tile table: out[c] = the first tile that starts in
// chunk c, out[n_chunks] = n_tiles; false if some chunk holds no tile.
bool chunk_segments(const std::vector<Tile> &tiles, int64_t n_chunks, std::vector<int32_t> *out);
// Waves per block of the separate sync for K workers (0: K takes the loop kernel).
int average_tile_waves(int K);
constexpr int kLdsPerCU = 160 * 1024;
// Resident waves per CU that the separate sync is timed with at init.
constexpr int kAverageCapWaves = 24;

// Record of one measurement (or, in a launch that the device ended without one,
// of the launch, in its first slot).
struct SlotHdr {
    int64_t t;        // the measured step (the launch's last without a measurement)
    int32_t due;      // 1: a sync followed the step
    int32_t p;        // period in force for the step (p, p_next, C2 and nC2: with the controller
    int32_t p_next;   // on the device, else 0), and after the sync's decision
    int32_t status;   // ADPSGD_OK, or ADPSGD_ENONFINITE when S was not finite
    double S;         // sum over tensors of the variances (0 without a measurement)
    double GN;        // sum over tensors of the gradient norms^2
    double C2;        // controller state after the step
    int64_t nC2;
    int32_t n;        // steps of the launch
    int32_t pad_;
};
constexpr size_t kSlotHdrBytes = 64;
static_assert(sizeof(SlotHdr) <= kSlotHdrBytes, "slot header");

struct ReduceParams {
    const double *tile_partials;  // [n_slots][2 n_tiles] (tile_stride apart)
    const Chunk *chunks;          // [n_chunks], in tensor order
    const int32_t *chunk_begin;   // [T + 1]: chunks of tensor tau
    double *chunk_partials;       // [n_slots][2 n_chunks] (chunk_stride apart)
    double *acc;                  // [n_slots][2T] device scratch: per-tensor sums
    double *sums;                 // [n_slots][2] device scratch: S, the norm total
    int64_t tile_stride, chunk_stride;   // doubles
    const int32_t *large;         // [n_large] tensors of more than kSmallTensorChunks chunks
    int32_t n_chunks, T, K, n_large;
    int32_t chunks_are_tiles;     // 1: chunk_partials is tile_partials (one tile per chunk)
    int32_t block0;               // first block of this launch of the chunk sums (set by launch_reduce)
    // More chunk partials than one LDS window: the tensors are cut into
    // windows (a run of whole small tensors whose chunks fit one window, or one
    // large tensor), reduced by one block each; the finishing block then sums
    // the window partials.  n_windows = 0: one block does everything.
    const int32_t *win_begin;     // [n_windows + 1]: first tensor of each window
    double *win_partials;         // [n_slots][2 n_windows]: per window, sum of variances, of gradient norms^2
    int32_t n_windows;
    int32_t n_slots;              // measurements of the launch at most, one record each
    // Records (header, then the variances and gradient norms^2 per tensor) in
    // host memory: slots slot0, slot0 + 1, ... of a ring, slot_bytes apart.
    char *recs;
    int64_t slot_bytes;
    int32_t slot0, ring;
    SchedState *sched;            // the controller state (when.device or control)
    int32_t control;              // 1: decisions are taken here and the state is kept up
    int32_t pad_;
    SchedRule rule;
    SpanWhen when;                // as in the launch that is reduced
    double gamma[kSpanSteps];     // rates in fp64 (Algorithm 2's gamma_t) from step when.t on
};

// Segmented fixed-order sums of the tile partials (chunks, then tensors, then
// over tensors) of every measurement of a launch and, with control, Algorithm
// 2's period decisions on the results, in step order.
// Windows of tensors (ReduceParams::win_begin) are cut by the host:
int32_t reduce_windows(int32_t T, const int32_t *chunk_begin, std::vector<int32_t> *win_begin);
hipError_t launch_reduce(const ReduceParams &r, hipStream_t st);
// Zero elements [0, P) of each of the K rows of a (rows ld apart); vec: ld is
// a multiple of 4 and a 16-byte aligned, so whole groups take one store.
hipError_t launch_zero_rows(float *a, int64_t ld, int64_t P, int32_t K, bool vec, hipStream_t st);
// Copy row 0's elements [0, P) to the other K - 1 rows.
hipError_t launch_spread_row(float *a, int64_t ld, int64_t P, int32_t K, bool vec, hipStream_t st);
hipError_t launch_init_problem(float *h, float *xs, int64_t P, uint64_t seed, double h_lo,
                               double h_hi, hipStream_t st);
hipError_t launch_philox_dump(uint64_t seed, uint32_t c1, uint32_t c2, uint32_t c3, int64_t g0,
                              int64_t n, uint32_t *out, hipStream_t st);
hipError_t launch_normal_dump(uint64_t seed, uint32_t c1, uint32_t c2, uint32_t c3, int64_t g0,
                              int64_t n, float *out, hipStream_t st);

}  // namespace adpsgd
