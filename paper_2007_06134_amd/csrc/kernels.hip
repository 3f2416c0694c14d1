// gfx950 kernels of the ADPSGD hot path.
//
//   k_local_step   1 to 64 local steps of every worker (Algorithm 2's update) in
//                  one streaming pass over x and m, with the noisy quadratic
//                  gradient generated in registers.
//   k_span         1 to 64 steps with the synchronizations among them (Algorithm
//                  2: replica mean, broadcast, per-element squared deviations,
//                  the parameter variance of Section II-B) on one aligned chunk
//                  of 256 elements, in one pass over x and m (K up to 128).
//   k_average      the synchronization alone (K up to 128 but 3).
//   k_sync_loop    one step with a sync for K above 128; the sync alone there and
//                  at K = 3.
//   k_reduce_chunks,  fixed-order sums of the tile partials per chunk, then
//   k_reduce_windows  per tensor (in windows of tensors when there are more
//   k_reduce_finish   chunk partials than one block's LDS holds) and over
//   k_control         tensors, for every sync of a launch at once, and Algorithm
//                     2's period decisions when a run's schedule lives on the
//                     device.
//   k_init_problem, k_zero_rows, k_philox_dump, k_normal_dump: problem data,
//                  row clearing and the raw generator streams.
//
// Work unit: a group of four consecutive elements of one worker's row, moved
// with one dwordx4 load and store and fed by one Philox call.  On MI355X a
// stream of one dwordx4 access per thread over a large grid sustains far more
// HBM bandwidth than threads that each walk many rows, so every thread of the
// local step owns a single (group, worker) pair.  At a sync the waves of a
// tile's block own the K rows and exchange their row sums through LDS.  No
// atomics and fixed reduction orders make results bit-reproducible for a
// given (K, P, offsets).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kernels.hpp"

namespace adpsgd {

namespace {

// Bring the first BYTES of the kernel's arguments into the scalar cache in one
// round trip, for a kernel of one block whose time is such round trips: read
// batch after batch where they are used, they cost k_reduce_finish 4.2 us
// instead of 3.5 (T = 1, 256 tiles).  The other kernels gain nothing by it.
template <int BYTES>
__device__ __forceinline__ void fetch_args() {
    const auto *args = (const __attribute__((address_space(4))) uint32_t *)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t line[BYTES / 64 + 1];
#pragma unroll
    for (int i = 0; i <= BYTES / 64; ++i) line[i] = args[i < BYTES / 64 ? 16 * i : BYTES / 4 - 1];
#pragma unroll
    for (int i = 0; i <= BYTES / 64; ++i) asm volatile("" ::"s"(line[i]));
}

__device__ __forceinline__ f4 fma4(f4 a, f4 b, f4 c) {
    return f4{fmaf(a.x, b.x, c.x), fmaf(a.y, b.y, c.y), fmaf(a.z, b.z, c.z), fmaf(a.w, b.w, c.w)};
}
__device__ __forceinline__ f4 splat(float v) { return f4{v, v, v, v}; }
// v, of which the compiler knows nothing.
__device__ __forceinline__ f4 opaque(f4 v) {
    float a = v.x, b = v.y, c = v.z, d = v.w;
    asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
    return f4{a, b, c, d};
}

// Replica rows are touched once per step and never reused before the next
// step, so with a working set beyond the on-chip caches they are streamed with
// non-temporal loads and stores.
template <bool NT>
__device__ __forceinline__ f4 ld4(const float *p) {
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p));
    else return *reinterpret_cast<const f4 *>(p);
}
template <bool NT>
__device__ __forceinline__ void st4(float *p, f4 v) {
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<f4 *>(p));
    else *reinterpret_cast<f4 *>(p) = v;
}

// Masked scalar access to the lanes of a group that lie in [lo, hi).
__device__ __forceinline__ bool in(int64_t e, int64_t lo, int64_t hi) { return e >= lo && e < hi; }
__device__ __forceinline__ f4 ld4_masked(const float *base, int64_t e0, int64_t lo, int64_t hi) {
    f4 v = splat(0.0f);
    if (in(e0 + 0, lo, hi)) v.x = base[0];
    if (in(e0 + 1, lo, hi)) v.y = base[1];
    if (in(e0 + 2, lo, hi)) v.z = base[2];
    if (in(e0 + 3, lo, hi)) v.w = base[3];
    return v;
}
__device__ __forceinline__ void st4_masked(float *base, f4 v, int64_t e0, int64_t lo, int64_t hi) {
    if (in(e0 + 0, lo, hi)) base[0] = v.x;
    if (in(e0 + 1, lo, hi)) base[1] = v.y;
    if (in(e0 + 2, lo, hi)) base[2] = v.z;
    if (in(e0 + 3, lo, hi)) base[3] = v.w;
}
__device__ __forceinline__ f4 mask4(f4 v, int64_t e0, int64_t lo, int64_t hi) {
    return f4{in(e0 + 0, lo, hi) ? v.x : 0.0f, in(e0 + 1, lo, hi) ? v.y : 0.0f,
              in(e0 + 2, lo, hi) ? v.z : 0.0f, in(e0 + 3, lo, hi) ? v.w : 0.0f};
}

// What a lane keeps of its group over workers and steps.  The gradient without
// its noise, h (x - x*) + wd x, is taken as hw (x - c) + b with hw = h + wd and
// (c, b) = (x*, wd x*) where |h| >= wd, else (0, -h x*): whichever is the larger of
// h and wd multiplies what it multiplies in the plain form, so each of the two terms
// is at most twice the larger of the plain form's and nothing cancels that does not
// cancel there.  (With (x*, wd x*) throughout, x after 200 steps at wd = 1, h = 1e-3
// is 5.3e-5 off in the 2-norm, 830 times the plain form's error; so chosen,
// 1.0 to 1.3 times it at every wd / h from 1e-3 to 1e8.)
template <int ROUNDS>
struct GroupData {
    f4 hw, c, b;
    PhiloxGroup pg;
    NoiseKeys<ROUNDS> keys;
    float sigma_r, mu;   // of the launch, in vector registers
};
template <int ROUNDS>
__device__ __forceinline__ GroupData<ROUNDS> group_data(const StepParams &a, int64_t g, f4 h, f4 xs) {
    f4 hw = h + splat(a.wd), c = xs, b = splat(a.wd) * xs;
    // (one test for the wave, where few problems need the other form: with a select for
    // every element 76 launches of one or two steps, K = 8, P = 11.2M, take 1.3% longer)
    if (__any(fminf(fminf(fabsf(h.x), fabsf(h.y)), fminf(fabsf(h.z), fabsf(h.w))) < a.wd)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool flat = fabsf(h[i]) < a.wd;
            c[i] = flat ? 0.0f : c[i];
            b[i] = flat ? -h[i] * xs[i] : b[i];
        }
    }
    // Four consecutive registers each, as loaded: scattered over the register file the
    // same instructions run 5% slower (32 steps at K = 8, P = 138M 22.0 ms, not 20.9).
    // With eight rows a wave at K = 32 (ROUNDS = 4), where registers are short, only c: 400
    // steps at P = 1.2M 9.51 ms, and 9.91 with all three.
    if constexpr (ROUNDS == 4) asm("" : "+v"(c));
    else asm("" : "+v"(hw), "+v"(c), "+v"(b));
    return GroupData<ROUNDS>{hw, c, b, philox_group((uint32_t)g, a.rk),
                             noise_keys<ROUNDS>(a.rk), in_vgpr(a.sigma_r), in_vgpr(a.mu)};
}
// The gradient of F(x) = 1/2 sum h (x - x*)^2 + wd/2 |x|^2.
template <int ROUNDS>
__device__ __forceinline__ f4 gradient(const GroupData<ROUNDS> &gd, f4 x) {
    return fma4(gd.hw, x - gd.c, gd.b);
}

// v = mu v + d in v's own register: left to itself the compiler adds into d's, and
// copies all of m in every step of a loop.
__device__ __forceinline__ float scale_add(float v, float mu, float d) {
    asm("v_fma_f32 %0, %0, %1, %2" : "+v"(v) : "v"(mu), "v"(d));
    return v;
}

// Step t + j of worker k: momentum SGD on the noisy quadratic, PyTorch-SGD form
// with coupled weight decay, d = h (x - x*) + sigma z + wd x;  m = mu m + d;
// x = x - gamma m.  d is taken as hw (x - c) + (b + sigma z) (GroupData): five
// operations an element instead of seven.  k is uniform over the wave.  Explicit
// fmaf fixes the rounding so every kernel computes identical bits.
// 64 steps at K = 16, P = 25.6M (k_local_step) take 10.7 ms; with the uniform
// operands in scalar registers, conversions to float and m copied, 11.9.
template <int ROUNDS>
__device__ __forceinline__ void sgd_step(const StepParams &a, const GroupData<ROUNDS> &gd, int k, f4 &x, f4 &m, int j = 0) {
    const u4 r = philox_noise(gd.pg, (uint32_t)k, a.t + (uint32_t)j, a.rk, gd.keys);
    const f4 d = fma4(gd.hw, x - gd.c, add_noise4(gd.sigma_r, r, gd.b));
    m = f4{scale_add(m.x, gd.mu, d.x), scale_add(m.y, gd.mu, d.y), scale_add(m.z, gd.mu, d.z), scale_add(m.w, gd.mu, d.w)};
    x = fma4(splat(in_vgpr(-a.gamma[j])), m, x);
}

// Sum of the squares of v's elements, in fp64.
__device__ __forceinline__ double square_sum(f4 v) {
    double q = (double)v.x * (double)v.x;
    q = fma((double)v.y, (double)v.y, q);
    q = fma((double)v.z, (double)v.z, q);
    return fma((double)v.w, (double)v.w, q);
}

// Sums of a pair of values over the block in a fixed order: wave64 butterfly,
// then the waves in order.  Valid on thread 0.  TWO = false: b is known to be
// zero everywhere (no gradient norm outside tracing) and is not reduced.
struct Pair {
    double a, b;
};
template <int WAVES, bool TWO = true>
__device__ __forceinline__ Pair block_sum2(double a, double b) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        if (TWO) b += __shfl_xor(b, off, 64);
    }
    if constexpr (WAVES == 1) {
        return Pair{a, TWO ? b : 0.0};
    } else {
        __shared__ double wave_a[WAVES], wave_b[TWO ? WAVES : 1];
        if ((threadIdx.x & 63) == 0) {
            wave_a[threadIdx.x >> 6] = a;
            if (TWO) wave_b[threadIdx.x >> 6] = b;
        }
        __syncthreads();
        Pair total{0.0, 0.0};
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                total.a += wave_a[w];
                if (TWO) total.b += wave_b[w];
            }
        }
        return total;
    }
}

// ---------------------------------------------------------------- local step

// Thread = (group g, worker k); a block covers BS consecutive groups (a
// chunk) of one worker's row.  Workgroups go round-robin over the 8 XCDs, and
// the blocks are ordered so that the K blocks of a chunk run on the same XCD:
// h and x* of the chunk come from HBM once and from that XCD's L2 for the
// other K-1 workers.  Within an XCD, S = row_chunks chunks of one worker's
// row come one after another, then the same S chunks of the next worker's
// row, so each row is streamed in runs of S chunks (S = 1: the K workers of
// one chunk in turn).  The best BS, S and LDS reservation depend on the shape
// and the machine; the runtime times a few.
// TAIL: P is not a multiple of 4, so the last group of every row is partial.
// n steps per launch: a step couples no two elements, so x and m stay in
// registers for all n and cross HBM once.  One step is bound by HBM, eight by
// arithmetic: at K = 8, P = 138M 1 / 2 / 4 / 8 / 16 steps take 2.97 / 3.01 /
// 3.27 / 5.07 / 8.78 ms, against 2.97 ms for each when launched one by one.
template <int BS, bool VEC, bool NT, bool TAIL>
__global__ void __launch_bounds__(BS) k_local_step(StepParams a) {
    const int64_t b = a.block0 + blockIdx.x;
    const int64_t s = b >> 3;                        // position within the XCD
    const int64_t run = s / a.row_chunks;            // (super-chunk, worker)
    const int k = (int)(run % a.K);
    const int64_t chunk = ((run / a.K) * a.row_chunks + (s - run * a.row_chunks)) * 8 + (b & 7);
    const int64_t g = chunk * BS + threadIdx.x;
    if (g >= a.n_groups) return;
    const int64_t e0 = 4 * g;
    float *xr = a.x + (int64_t)k * a.ld + e0;
    float *mr = a.m + (int64_t)k * a.ld + e0;
    if (VEC && (!TAIL || e0 + 4 <= a.P)) {
        f4 x = ld4<NT>(xr), m = ld4<NT>(mr);
        const f4 h = ld4<false>(a.h + e0), xs = ld4<false>(a.xs + e0);
        const auto gd = group_data<8>(a, g, h, xs);
#pragma unroll 1
        for (int j = 0; j < a.n; ++j) sgd_step(a, gd, k, x, m, j);
        st4<NT>(xr, x);
        st4<NT>(mr, m);
    } else {
        // the ragged last group of a row, or rows that are not 16-byte aligned
        // (a row stride that is not a multiple of 4): scalar accesses, masked
        // to [0, P)
        f4 x = ld4_masked(xr, e0, 0, a.P), m = ld4_masked(mr, e0, 0, a.P);
        const f4 h = ld4_masked(a.h + e0, e0, 0, a.P), xs = ld4_masked(a.xs + e0, e0, 0, a.P);
        const auto gd = group_data<8>(a, g, h, xs);
#pragma unroll 1
        for (int j = 0; j < a.n; ++j) sgd_step(a, gd, k, x, m, j);
        st4_masked(xr, x, e0, 0, a.P);
        st4_masked(mr, m, e0, 0, a.P);
    }
}

// ---------------------------------------------------------------- sync

// Pairwise sum of rows[base .. base+N) at one lane, in a fixed tree order (left
// half, right half).  Exact when all rows are equal and N is a power of two,
// so a sync right after a sync leaves zero variance.  Depth-first evaluation
// keeps only O(log N) partial sums live.
template <int N>
__device__ __forceinline__ f4 tree_sum_lds(const f4 (*rows)[64], int lane, int base) {
    if constexpr (N == 1) {
        return rows[base][lane];
    } else {
        const f4 l = tree_sum_lds<N / 2>(rows, lane, base);
        const f4 r = tree_sum_lds<N - N / 2>(rows, lane, base + N / 2);
        return l + r;
    }
}

// The same tree over a thread's own registers v[base .. base+N).  For N and K
// powers of two, rows R w .. R w + R - 1 form one node of the K-row tree, so
// summing a wave's R rows here and the W node sums through LDS gives the same
// bits as the K-row tree.
template <int N>
__device__ __forceinline__ f4 tree_sum_regs(const f4 *v, int base) {
    if constexpr (N == 1) {
        return v[base];
    } else {
        return tree_sum_regs<N / 2>(v, base) + tree_sum_regs<N - N / 2>(v, base + N / 2);
    }
}

// The pairwise tree over a run-time number (1 to 16) of LDS entries.
__device__ __forceinline__ f4 tree_sum_lds_n(const f4 (*rows)[64], int lane, int n) {
    switch (n) {
    case 1: return tree_sum_lds<1>(rows, lane, 0);
    case 2: return tree_sum_lds<2>(rows, lane, 0);
    case 3: return tree_sum_lds<3>(rows, lane, 0);
    case 4: return tree_sum_lds<4>(rows, lane, 0);
    case 5: return tree_sum_lds<5>(rows, lane, 0);
    case 6: return tree_sum_lds<6>(rows, lane, 0);
    case 7: return tree_sum_lds<7>(rows, lane, 0);
    case 8: return tree_sum_lds<8>(rows, lane, 0);
    case 9: return tree_sum_lds<9>(rows, lane, 0);
    case 10: return tree_sum_lds<10>(rows, lane, 0);
    case 11: return tree_sum_lds<11>(rows, lane, 0);
    case 12: return tree_sum_lds<12>(rows, lane, 0);
    case 13: return tree_sum_lds<13>(rows, lane, 0);
    case 14: return tree_sum_lds<14>(rows, lane, 0);
    case 15: return tree_sum_lds<15>(rows, lane, 0);
    default: return tree_sum_lds<16>(rows, lane, 0);
    }
}

// The replica mean at one lane from the W wave sums in LDS: the pairwise tree
// (WC = W waves for a compiled K, else W from K), so that with R rows per wave
// the mean is the K-row tree when K is a power of two and exact for equal
// replicas; with one row per wave (RD = 1, K = 3) the rows in row order, as
// the loop kernel adds them.
template <int KT, int WC, int RD>
__device__ __forceinline__ f4 lds_mean(const f4 (*rows)[64], int lane, int W, int K) {
    if constexpr (KT > 0) {
        // every compiled K is a power of two: the product by 1/K is the
        // correctly rounded quotient, the same bits as the division, at a
        // fraction of its instructions
        static_assert((KT & (KT - 1)) == 0, "compiled worker counts are powers of two");
        return tree_sum_lds<WC>(rows, lane, 0) * splat(1.0f / (float)KT);
    } else if constexpr (RD > 1) {
        return tree_sum_lds_n(rows, lane, W) / splat((float)K);
    } else {
        // the reads go out four at a time, and the adds run in wave order
        f4 s = rows[0][lane];
#pragma unroll 1
        for (int w0 = 1; w0 < W; w0 += 4) {
            f4 v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = w0 + j < W ? rows[w0 + j][lane] : splat(0.0f);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (w0 + j < W) s = s + v[j];
        }
        return s / splat((float)K);
    }
}

__device__ __forceinline__ f4 shfl_xor4(f4 v, int off) {
    return f4{__shfl_xor(v.x, off, 64), __shfl_xor(v.y, off, 64), __shfl_xor(v.z, off, 64), __shfl_xor(v.w, off, 64)};
}

// The replica mean of every group of a tile from the W wave sums in LDS,
// formed once per group instead of by every wave: wave w takes groups
// w G .. w G + G - 1 (G = 64 / W), its lane l the wave sum l % W of group
// w G + l / W, and a butterfly over those W lanes adds them as the pairwise
// tree does (each pair in the tree's order up to commutation, so the same bits
// as tree_sum_lds<W>).  The means of the first n groups go to out[64]; callers
// put a barrier before (the wave sums) and after (the means).  For a block of
// 16 waves this reads 1/16 of the LDS that every wave reading all 16 sums
// reads (1-2% of the separate sync at K = 32).
template <int W, int KT>
__device__ __forceinline__ void group_means(const f4 (*sums)[64], f4 *out, int lane, int w, int n) {
    static_assert((W & (W - 1)) == 0 && (KT & (KT - 1)) == 0, "power-of-two waves and workers");
    constexpr int G = 64 / W;
    const int j = w * G + lane / W, i = lane % W;
    f4 v = j < n ? sums[i][j] : splat(0.0f);
#pragma unroll
    for (int off = 1; off < W; off <<= 1) v = v + shfl_xor4(v, off);
    if (i == 0) out[j] = v * splat(1.0f / (float)KT);
}

// block_sum2 over a run-time number of waves (at most 16), in the same order.
template <bool TWO = true>
__device__ __forceinline__ Pair block_sum2_waves(double a, double b, int waves) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        if (TWO) b += __shfl_xor(b, off, 64);
    }
    __shared__ double wave_a[16], wave_b[TWO ? 16 : 1];
    if ((threadIdx.x & 63) == 0) {
        wave_a[threadIdx.x >> 6] = a;
        if (TWO) wave_b[threadIdx.x >> 6] = b;
    }
    __syncthreads();
    Pair total{0.0, 0.0};
    if (threadIdx.x == 0)
        for (int w = 0; w < waves; ++w) {
            total.a += wave_a[w];
            if (TWO) total.b += wave_b[w];
        }
    return total;
}

// Waves per block of the separate sync: with no step to take, two rows per wave
// beat one (+2 to +15%).  KT = 0: K is a kernel argument (a K up to 128 without
// a compiled variant, with RD = 2, 4 or 8 rows per wave); 16 is the most waves
// such a block has.
template <int KT>
constexpr int average_waves() {
    if constexpr (KT == 0) return 16;
    else if constexpr (KT >= 2) return KT / 2 < 16 ? KT / 2 : 16;
    else return 1;
}

// The separate sync of one aligned chunk of 256 elements (at most 64 groups, one
// per lane).  Wave w owns the rows k = R w .. R w + R - 1: it publishes their
// pairwise sum in LDS, reads the W sums of its lane back to form the mean in a
// fixed order (the same bits in every thread, and the same as a tree over all
// K rows), sums its squared deviations and writes the mean over its rows (with
// averaged momentum, the momentum rows too).  partials[2 tile] = the sum of
// squared deviations of each tile of the chunk.  Lanes of groups cut by the
// chunk's end use masked scalar accesses.  RAGGED (K an argument, K not a
// multiple of RD): the last wave holds fewer rows; the missing ones count as
// zeros in its sum.
template <int KT, bool VEC, bool NT, bool AVGM, int RD = 0, bool RAGGED = false>
__global__ void __launch_bounds__(64 * average_waves<KT>()) k_average(SyncParams p) {
    static_assert((KT == 0) == (RD > 0), "RD (rows per wave) is given exactly when K is an argument");
    static_assert(!RAGGED || RD >= 2, "a ragged last wave comes with several rows per wave");
    constexpr int WMAX = average_waves<KT>();
    constexpr int R = KT > 0 ? KT / WMAX : RD;
    const int W = KT > 0 ? WMAX : (p.s.K + (RD > 0 ? RD : 1) - 1) / (RD > 0 ? RD : 1);
    // a block of 16 waves forms each group's mean once (group_means)
    constexpr bool SPLIT = KT > 0 && WMAX >= 16;
    // wave w owns rows R w .. R w + R - 1 and publishes their subtree sum
    __shared__ f4 part[WMAX][64];
    __shared__ f4 mpart[AVGM ? WMAX : 1][64];
    __shared__ f4 means[SPLIT ? 64 : 1], mmeans[SPLIT && AVGM ? 64 : 1];
    const StepParams &a = p.s;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // the block's aligned chunk and its tiles (one per tensor in it)
    const int64_t c = p.s.block0 + blockIdx.x;
    const int64_t lo = c * kTileElems, hi = lo + kTileElems < a.P ? lo + kTileElems : a.P;
    // The chunk's first tile and the next chunk's.  Blocks of 16 waves read
    // them as scalars here; smaller blocks load them in lanes 0 and 1 (a
    // vector load, so that no wait for them comes ahead of the row loads) and
    // take them after the barrier.
    constexpr bool SEG_VEC = WMAX < 16;
    int32_t s0 = 0, s1 = 0, seg_l = 0;
    if constexpr (SEG_VEC) {
        seg_l = p.chunk_seg[c + (lane & 1)];
    } else {
        s0 = p.chunk_seg[c];
        s1 = p.chunk_seg[c + 1];
    }
    const int64_t e0 = 4 * ((lo >> 2) + lane);
    const bool active = e0 < hi;
    const bool full = VEC && e0 + 4 <= hi;
    // row R w + r exists (only the last wave's last rows can be missing)
    bool has[R];
#pragma unroll
    for (int r = 0; r < R; ++r) has[r] = !RAGGED || R * w + r < a.K;
    f4 xr[R];
    if (active) {
        f4 m[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            xr[r] = splat(0.0f);
            m[r] = splat(0.0f);
            if (!has[r]) continue;
            const float *xrow = a.x + (int64_t)(R * w + r) * a.ld + e0;
            xr[r] = full ? ld4<NT>(xrow) : ld4_masked(xrow, e0, lo, hi);
            if (AVGM) {
                const float *mrow = a.m + (int64_t)(R * w + r) * a.ld + e0;
                m[r] = full ? ld4<NT>(mrow) : ld4_masked(mrow, e0, lo, hi);
            }
        }
        part[w][lane] = tree_sum_regs<R>(xr, 0);   // (rows a ragged last wave lacks hold zeros)
        if (AVGM) mpart[w][lane] = tree_sum_regs<R>(m, 0);
    }
    __syncthreads();
    if constexpr (SEG_VEC) {
        s0 = __builtin_amdgcn_readlane(seg_l, 0);
        s1 = __builtin_amdgcn_readlane(seg_l, 1);
    }
    const bool one_tile = s1 - s0 == 1;   // uniform over the block
    if constexpr (SPLIT) {
        // groups of the chunk with elements in [lo, hi): the lanes that stored a sum
        const int64_t n64 = (hi - lo + 3) / 4;
        const int n = n64 < 64 ? (int)n64 : 64;
        group_means<WMAX, KT>(part, means, lane, w, n);
        if (AVGM) group_means<WMAX, KT>(mpart, mmeans, lane, w, n);
        __syncthreads();
    }
    // a chunk of one tile sums its squared deviations per row; a chunk of
    // several keeps them per element (over the rows), to split them by tile
    double acc = 0.0;
    double acc4[4] = {0.0, 0.0, 0.0, 0.0};
    if (active) {
        f4 mean;
        if constexpr (SPLIT) mean = means[lane];
        else mean = lds_mean<KT, WMAX, RD>(part, lane, W, a.K);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!has[r]) continue;
            f4 d = mean - xr[r];
            if (!full) d = mask4(d, e0, lo, hi);
            if (one_tile) {
                acc += square_sum(d);
            } else {
                acc4[0] = fma((double)d.x, (double)d.x, acc4[0]);
                acc4[1] = fma((double)d.y, (double)d.y, acc4[1]);
                acc4[2] = fma((double)d.z, (double)d.z, acc4[2]);
                acc4[3] = fma((double)d.w, (double)d.w, acc4[3]);
            }
            float *xrow = a.x + (int64_t)(R * w + r) * a.ld + e0;
            if (full) st4<NT>(xrow, mean); else st4_masked(xrow, mean, e0, lo, hi);
        }
        if (AVGM) {
            f4 mmean;
            if constexpr (SPLIT) mmean = mmeans[lane];
            else mmean = lds_mean<KT, WMAX, RD>(mpart, lane, W, a.K);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!has[r]) continue;
                float *mrow = a.m + (int64_t)(R * w + r) * a.ld + e0;
                if (full) st4<NT>(mrow, mmean); else st4_masked(mrow, mmean, e0, lo, hi);
            }
        }
    }
    if (one_tile) {
        Pair total;
        if constexpr (KT > 0) total = block_sum2<WMAX, false>(acc, 0.0);
        else total = block_sum2_waves<false>(acc, 0.0, W);
        if (threadIdx.x == 0) {
            p.partials[2 * s0] = total.a;
            p.partials[2 * s0 + 1] = 0.0;
        }
        return;
    }
    // several tiles (tensors) in the chunk: one fixed-order block sum each, of
    // the elements in its range
    for (int32_t sgi = s0; sgi < s1; ++sgi) {
        const Tile t = p.tiles[sgi];
        double v = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (in(e0 + j, t.start, t.start + t.len)) v += acc4[j];
        Pair total;
        if constexpr (KT > 0) total = block_sum2<WMAX, false>(v, 0.0);
        else total = block_sum2_waves<false>(v, 0.0, W);
        if (threadIdx.x == 0) {
            p.partials[2 * sgi] = total.a;
            p.partials[2 * sgi + 1] = 0.0;
        }
        __syncthreads();   // the block sum's LDS is used again for the next tile
    }
}

// ---------------------------------------------------------------- spans

// Sum over the wave, in every lane: lanes i and i ^ 1, then i ^ 2, quads and
// rows of 16 by mirroring (the same pairs of sums as i ^ 4 and i ^ 8), then the
// row and half swaps.  All 64 lanes take part.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v = dpp_add<0x141>(v);   // row_half_mirror
    v = dpp_add<0x140>(v);   // row_mirror
    {
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
        v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    }
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// A whole group of a row that is 16-byte aligned (VEC) or only as its elements are:
// global memory takes dwordx4 accesses at any multiple of four bytes, in place of
// four that each touch all of a wave's kilobyte.  A step with its sync, packed rows of
// 100M elements in all, with four single accesses and so: K = 8 587 and 358 us, K = 48
// 688 and 415 (with one step a launch 643 and 559).
typedef float f4_unaligned __attribute__((ext_vector_type(4), aligned(4)));
template <bool VEC, bool NT>
__device__ __forceinline__ f4 ld_group(const float *p) {
    if constexpr (VEC) return ld4<NT>(p);
    else return *reinterpret_cast<const f4_unaligned *>(p);
}
template <bool VEC, bool NT>
__device__ __forceinline__ void st_group(float *p, f4 v) {
    if constexpr (VEC) st4<NT>(p, v);
    else *reinterpret_cast<f4_unaligned *>(p) = v;
}

// Access to the first `left` elements of a group (at most 4; none when left <= 0).
__device__ __forceinline__ f4 ld4_left(const float *base, int left) {
    f4 v = splat(0.0f);
    if (left > 0) v.x = base[0];
    if (left > 1) v.y = base[1];
    if (left > 2) v.z = base[2];
    if (left > 3) v.w = base[3];
    return v;
}
__device__ __forceinline__ void st4_left(float *base, f4 v, int left) {
    if (left > 0) base[0] = v.x;
    if (left > 1) base[1] = v.y;
    if (left > 2) base[2] = v.z;
    if (left > 3) base[3] = v.w;
}
// v's elements first + i that lie in [begin, begin + len), the others zero.
__device__ __forceinline__ f4 mask4_range(f4 v, int first, int begin, int len) {
    const uint32_t i = (uint32_t)(first - begin), n = (uint32_t)len;
    return f4{i < n ? v.x : 0.0f, i + 1 < n ? v.y : 0.0f, i + 2 < n ? v.z : 0.0f, i + 3 < n ? v.w : 0.0f};
}

template <int N>
__device__ __forceinline__ double tree_sum_regs_d(const double *v, int base) {
    if constexpr (N == 1) return v[base];
    else return tree_sum_regs_d<N / 2>(v, base) + tree_sum_regs_d<N - N / 2>(v, base + N / 2);
}
template <int N>
__device__ __forceinline__ double tree_sum_lds_d(const double (*rows)[64], int lane, int base) {
    if constexpr (N == 1) {
        return rows[base][lane];
    } else {
        const double l = tree_sum_lds_d<N / 2>(rows, lane, base);
        const double r = tree_sum_lds_d<N - N / 2>(rows, lane, base + N / 2);
        return l + r;
    }
}

// With K an argument a block has up to 16 waves.  A CU deals a block's waves out to
// its four SIMDs, the first getting one more where they do not divide, so it holds
// two blocks of up to 12 waves when six waves' registers fit a SIMD (FEW), and two
// of 13 to 16 only when eight's do.
constexpr int kFewWaves = 12;

// Waves per block of k_span with R rows per wave, at most.
template <int KT, int R, bool FEW>
constexpr int span_waves() {
    if constexpr (KT == 0) return FEW ? kFewWaves : 16;
    else return KT / R;
}

// Philox rounds whose keys k_span keeps in vector registers.  What decides is the
// registers left: waves count for more than the keys do.  Measured with and
// without: 400 steps at K = 32, P = 1.2M (eight rows a wave) 9.1 and 9.7 ms with the
// keys of four rounds, but 32 steps at K = 8, P = 138M (eight rows, one wave a
// block) 21.7 and 20.5 ms, and 100 at K = 16, P = 25.6M (four rows) 22.9 and 22.5
// with one round's.  With one row a wave the launch is bound by HBM or by latency.
// Only 13 to 16 waves of four rows, one block a CU either way, have room for all (32
// steps at K = 56, 160M elements, 3.38 and 3.41 ms).
template <int KT, int R, bool FEW>
constexpr int span_vector_keys() {
    if constexpr (KT == 0) return R == 4 && !FEW ? 8 : 0;
    else if constexpr (KT == 1) return 8;
    else return KT == 32 && R == 8 ? 4 : 0;
}

// Waves per SIMD that k_span's registers leave room for, at least.  With K an
// argument they make room for two blocks a CU (some registers spill around a
// measurement, none in the steps).  One and two blocks, x of 160M elements, a step
// with its sync: K = 24 609 and 481 us, K = 28 617 and 561, K = 33 637 and 522; 32 steps
// in one launch: K = 24 3.27 and 2.62 ms, K = 31 3.20 and 2.74, K = 33 3.52 and 3.02.
template <int KT, int R, bool FEW>
constexpr int span_occupancy() {
    if constexpr (R == 1) return KT == 0 ? 6 : (KT == 1 ? 7 : 8);
    else if constexpr (R == 2) return KT == 0 ? (FEW ? 6 : 8) : (KT == 32 ? 8 : 7);
    else if constexpr (R == 4) return KT == 0 ? (FEW ? 6 : 4) : 5;
    else return 4;
}

// Several steps and the syncs among them on one aligned chunk of 256 elements
// (at most 64 groups, one per lane): a step couples no two elements and a sync
// only the K replicas of one, so x and m stay in registers for the whole span
// and cross HBM once.  Wave w owns the rows k = R w .. R w + R - 1.  After a
// step that a sync follows (or after every step when all are measured), the
// waves exchange their rows' pairwise sums through LDS, every thread forms the
// mean in a fixed order (see lds_mean), and the squared deviations are added
// over the rows pairwise and then over the lanes, by one wave of the block
// (each measurement another one, so that the extra work spreads over the
// SIMDs).  For a compiled K (a power of two) both sums are trees of which a
// wave's rows are a node, so every R gives the same bits.  The measurement of
// the span's j-th measured step goes to partials[j slot_stride + 2 tile + {0, 1}] =
// (sum of squared deviations, squared gradient norm at the mean; the latter
// only when every step is measured).
//
// Which steps a sync follows is planned by the host (when.syncs), or the span
// ends with the first step that Algorithm 2's counter, read from the device's
// controller state, says is due (when.device; span_plan).
//
// Bound: a span of one step by HBM, of five and more by vector arithmetic: a row's
// step is 68 to 73 instructions, among them 16 32-bit products (at least 4 cycles a
// wave) and 8 transcendental functions (8 cycles), at least 216 cycles of issue in all;
// at K = 8, P = 138M a SIMD issues one every 3.6 cycles, where these limits give 3.2.
// With the steps launched one by one, then in spans of two rows a wave, then so: 32
// steps at K = 8, P = 138M 96.8 / 25.4 / 21.1 ms, 24 traced at K = 8, P = 11.2M 6.41 /
// 1.94 / 1.50 ms.
template <int KT, int R, bool VEC, bool NT, bool FEW = false>
__global__ void __launch_bounds__((64 * span_waves<KT, R, FEW>()), (span_occupancy<KT, R, FEW>())) k_span(SpanParams p) {
    constexpr int WMAX = span_waves<KT, R, FEW>();
    const StepParams &a = p.s;
    const int K = KT > 0 ? KT : a.K;
    const int W = KT > 0 ? WMAX : (K + R - 1) / R;
    // blocks of 8 and 16 waves form each group's mean once (group_means)
    constexpr bool SPLIT = KT > 0 && WMAX >= 8;
    // part: the waves' sums of their rows; dev: of their squared deviations.  With K an
    // argument they take what the launch gives them (span_lds), W waves' worth: with room
    // for 16 a CU held six blocks of K = 3's three waves (a step with its sync, 160M
    // elements, 536 us; so 502).
    extern __shared__ f4 span_lds_base[];
    __shared__ f4 part_s[KT > 0 ? WMAX : 1][64];
    __shared__ f4 means[SPLIT ? 64 : 1];
    __shared__ double dev_s[KT > 0 ? WMAX : 1][64];
    auto part = [&](int i) -> f4 (&)[64] {
        if constexpr (KT > 0) return part_s[i];
        else return reinterpret_cast<f4 (*)[64]>(span_lds_base)[i];
    };
    auto dev = [&](int i) -> double (&)[64] {
        if constexpr (KT > 0) return dev_s[i];
        else return reinterpret_cast<double (*)[64]>(span_lds_base + 64 * W)[i];
    };
    const SpanPlan sp = span_plan(p.when, p.sched, p.rule);
    if (sp.n == 0) return;
    const int lane = threadIdx.x & 63;
    const int w = WMAX > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int64_t c = a.block0 + blockIdx.x;
    const int64_t lo = c * kTileElems, hi = lo + kTileElems < a.P ? lo + kTileElems : a.P;
    const int64_t g = (lo >> 2) + lane;
    const int e = 4 * lane;                // the lane's first element in the chunk
    const int len = (int)(hi - lo), left = len - e;
    // the whole chunk moves as float4 groups (uniform), or single lanes are cut
    const bool whole = len == (int)kTileElems;
    const bool full = VEC && left >= 4;
    bool has[R];   // row R w + r exists (uniform; only the last wave's last rows can be missing)
#pragma unroll
    for (int r = 0; r < R; ++r) has[r] = KT > 0 || R == 1 || R * w + r < K;
    // uniform row addresses (the lane's offset is 32 bits)
    float *const xb = a.x + (int64_t)(R * w) * a.ld + lo;
    float *const mb = a.m + (int64_t)(R * w) * a.ld + lo;
    // merged rows: row 0 for all, from the cache for all waves but one
    const bool x_one = sp.merged_in, m_one = sp.merged_in && p.avg_m;
    f4 x[R], m[R], h, xs;
    if (whole) {
        if constexpr (KT == 0) {
            // every load goes out before one is waited for, as a copied row is
            auto load_rows = [&](f4 *v, const float *rows, const float *row0, bool one) {
                if (one) {
                    const f4 v0 = ld_group<VEC, false>(row0 + e);
#pragma unroll
                    for (int r = 0; r < R; ++r) v[r] = has[r] ? v0 : splat(0.0f);
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) v[r] = has[r] ? ld_group<VEC, NT>(rows + r * a.ld + e) : splat(0.0f);
                }
            };
            h = ld4<false>(a.h + lo + e);
            xs = ld4<false>(a.xs + lo + e);
            load_rows(m, mb, a.m + lo, m_one);
            load_rows(x, xb, a.x + lo, x_one);
        } else {
            // (with one row a wave a CU's 32 waves have more loads out so than HBM
            // takes well: a step with its sync, K = 8, P = 20M, 459 us row by row, 494 so)
            if (x_one) x[0] = ld_group<VEC, false>(a.x + lo + e);
            if (m_one) m[0] = ld_group<VEC, false>(a.m + lo + e);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                x[r] = x_one ? x[0] : ld_group<VEC, NT>(xb + r * a.ld + e);
                m[r] = m_one ? m[0] : ld_group<VEC, NT>(mb + r * a.ld + e);
            }
            h = ld4<false>(a.h + lo + e);
            xs = ld4<false>(a.xs + lo + e);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            x[r] = m[r] = splat(0.0f);
            if (!has[r]) continue;
            const float *const xr = x_one ? a.x + lo + e : xb + r * a.ld + e;
            const float *const mr = m_one ? a.m + lo + e : mb + r * a.ld + e;
            x[r] = full ? ld4<NT>(xr) : ld4_left(xr, left);
            m[r] = full ? ld4<NT>(mr) : ld4_left(mr, left);
        }
        // (h and x* are aligned whatever the rows' stride)
        h = left >= 4 ? ld4<false>(a.h + lo + e) : ld4_left(a.h + lo + e, left);
        xs = left >= 4 ? ld4<false>(a.xs + lo + e) : ld4_left(a.xs + lo + e, left);
    }
    // the chunk's first tile and the next chunk's, in lanes 0 and 1: a vector
    // load, so that no wait for it comes ahead of the row loads
    const int32_t seg_l = p.chunk_seg[c + (lane & 1)];
    const auto gd = group_data<span_vector_keys<KT, R, FEW>()>(a, g, h, xs);
    const int j0 = (int)(sp.t - p.when.t);   // the first step's rate is gamma[j0]
    int slot = 0;
#pragma unroll 1
    for (int j = 0; j < sp.n; ++j) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (has[r]) sgd_step(a, gd, R * w + r, x[r], m[r], j0 + j);
        const bool due = (sp.syncs >> j) & 1;
        if (!due && !p.when.measure) continue;   // uniform over the block

        // the mean of the K rows v at every lane (part and means are free on entry)
        auto row_mean = [&](const f4 *v) -> f4 {
            if constexpr (WMAX == 1) return tree_sum_regs<R>(v, 0) * splat(1.0f / (float)KT);
            part(w)[lane] = tree_sum_regs<R>(v, 0);   // (rows a ragged last wave lacks hold zeros)
            __syncthreads();
            if constexpr (SPLIT) {
                group_means<WMAX, KT>(part_s, means, lane, w, 64);
                __syncthreads();
                return means[lane];
            }
            return lds_mean<KT, WMAX, R>(&part(0), lane, W, K);
        };
        const f4 mean = row_mean(x);
        if (due && p.avg_m) {
            if constexpr (WMAX > 1) __syncthreads();   // part and means are read
            const f4 mmean = row_mean(m);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (has[r]) m[r] = mmean;
        }
        const int32_t s0 = __builtin_amdgcn_readlane(seg_l, 0), s1 = __builtin_amdgcn_readlane(seg_l, 1);
        const bool summer = WMAX == 1 || w == (int)((uint32_t)(c + slot) % (uint32_t)W);
        double *const out = p.partials + (int64_t)slot * p.slot_stride;
        // the sums of the chunk's elements [begin, begin + n) (CUT: not all 256) for tile sgi
        auto tile_sums = [&](auto cut, int32_t sgi, int begin, int n) {
            constexpr bool CUT = decltype(cut)::value;
            // (opaque in a tile of several: the differences of all rows, formed once
            // for every tile, would not stay in registers)
            const f4 mean_t = CUT ? opaque(mean) : mean;
            double q[KT > 0 ? R : 1];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                f4 d = mean_t - x[r];
                if (CUT) d = mask4_range(d, e, begin, n);
                if constexpr (KT > 0) q[r] = square_sum(d);
                else if (r == 0) q[0] = square_sum(d);   // (every wave has a first row)
                else if (has[r]) q[0] += square_sum(d);
            }
            double v;
            if constexpr (KT > 0) v = tree_sum_regs_d<R>(q, 0);
            else v = q[0];
            if constexpr (WMAX > 1) {
                dev(w)[lane] = v;
                __syncthreads();
                if (summer) {
                    if constexpr (KT > 0) {
                        v = tree_sum_lds_d<WMAX>(dev_s, lane, 0);
                    } else {
                        v = dev(0)[lane];
                        for (int i = 1; i < W; ++i) v += dev(i)[lane];
                    }
                }
                if (CUT) __syncthreads();   // dev is read before the next tile's sums
            }
            if (summer) {
                v = wave_sum(v);
                double gn = 0.0;
                if (p.when.measure) {
                    f4 gr = gradient(gd, mean_t);
                    if (CUT) gr = mask4_range(gr, e, begin, n);
                    gn = wave_sum(square_sum(gr));
                }
                if (lane == 0) {
                    out[2 * (int64_t)sgi] = v;
                    out[2 * (int64_t)sgi + 1] = gn;
                }
            }
        };
        // one sum per tile (tensor) of the chunk; usually all of the chunk is one
        // (a path of its own: the masks of the others cost half as much again)
        if (s1 - s0 == 1 && len == (int)kTileElems) {
            tile_sums(std::false_type{}, s0, 0, (int)kTileElems);
        } else {
            for (int32_t sgi = s0; sgi < s1; ++sgi) {
                const Tile t = p.tiles[sgi];
                tile_sums(std::true_type{}, sgi, (int)(t.start - lo), t.len);
            }
        }
        if (due) {
            asm volatile("");   // (a branch, not a select for every element)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (has[r]) x[r] = mean;
        }
        ++slot;
    }
    if constexpr (WMAX > 1) {
        // every wave has read the merged row before one writes it (a measurement's
        // barriers, which come after the steps that used it, see to that too)
        if (sp.merged_in && sp.syncs == 0 && !p.when.measure) {
            asm volatile("" ::"v"(x[0].x), "v"(m[0].x));
            __syncthreads();
        }
    }
    // (row 0 alone where the launch leaves merged rows)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!has[r]) continue;
        const bool lead = R * w + r == 0;   // uniform
        const bool x_out = lead || !sp.merged_out, m_out = lead || !(sp.merged_out && p.avg_m);
        if (whole) {
            if (x_out) st_group<VEC, NT>(xb + r * a.ld + e, x[r]);
            if (m_out) st_group<VEC, NT>(mb + r * a.ld + e, m[r]);
        } else {
            if (x_out) { if (full) st4<NT>(xb + r * a.ld + e, x[r]); else st4_left(xb + r * a.ld + e, x[r], left); }
            if (m_out) { if (full) st4<NT>(mb + r * a.ld + e, m[r]); else st4_left(mb + r * a.ld + e, m[r], left); }
        }
    }
}

// K above 128 (and the separate sync at K = 3): one wave per tile, lane = group,
// the workers walked in a loop.  The first pass takes the span's one step (with
// STEP), stores the replicas and sums them; the second re-reads them for the
// deviations and, when a sync is due, writes the mean.  With averaged momentum
// the first pass also sums the momentum buffers and the second writes their
// mean.  A step that is neither synced nor measured is the first pass alone.
template <bool VEC, bool STEP>
__global__ void __launch_bounds__(64) k_sync_loop(SpanParams p) {
    const StepParams &a = p.s;
    bool bcast = true, measure = true;
    int j = 0;
    if constexpr (STEP) {
        const SpanPlan sp = span_plan(p.when, p.sched, p.rule);
        if (sp.n == 0) return;
        j = (int)(sp.t - p.when.t);
        bcast = sp.syncs & 1;
        measure = bcast || p.when.measure;
    }
    const bool grad = STEP && p.when.measure;
    const bool sum_m = p.avg_m, avg_m = sum_m && bcast;
    const int64_t ti = p.s.block0 + blockIdx.x;
    const Tile tile = p.tiles[ti];
    const int64_t lo = tile.start, hi = tile.start + tile.len;
    const int64_t g = (lo >> 2) + threadIdx.x;
    const int64_t e0 = 4 * g;
    double acc = 0.0, gn = 0.0;
    if (e0 < hi) {
        const bool full = VEC && e0 >= lo && e0 + 4 <= hi;
        f4 h = splat(0.0f), xs = splat(0.0f);
        if (STEP) {
            if (full) { h = ld4<false>(a.h + e0); xs = ld4<false>(a.xs + e0); }
            else { h = ld4_masked(a.h + e0, e0, lo, hi); xs = ld4_masked(a.xs + e0, e0, lo, hi); }
        }
        const auto gd = group_data<8>(a, g, h, xs);
        f4 s = splat(0.0f), sm = splat(0.0f);
        for (int k = 0; k < a.K; ++k) {
            float *xrow = a.x + (int64_t)k * a.ld + e0;
            float *mrow = a.m + (int64_t)k * a.ld + e0;
            f4 x = full ? ld4<false>(xrow) : ld4_masked(xrow, e0, lo, hi);
            f4 m = splat(0.0f);
            if (STEP || sum_m) m = full ? ld4<false>(mrow) : ld4_masked(mrow, e0, lo, hi);
            if (STEP) {
                sgd_step(a, gd, k, x, m, j);
                if (full) st4<false>(xrow, x); else st4_masked(xrow, x, e0, lo, hi);
                if (!avg_m) { if (full) st4<false>(mrow, m); else st4_masked(mrow, m, e0, lo, hi); }
            }
            s = (k == 0) ? x : s + x;
            if (sum_m) sm = (k == 0) ? m : sm + m;
        }
        if (measure) {
            const f4 mean = s / splat((float)a.K);
            const f4 mmean = sm / splat((float)a.K);
            for (int k = 0; k < a.K; ++k) {
                float *xrow = a.x + (int64_t)k * a.ld + e0;
                const f4 x = full ? ld4<false>(xrow) : ld4_masked(xrow, e0, lo, hi);
                f4 d = mean - x;
                if (!full) d = mask4(d, e0, lo, hi);
                acc += square_sum(d);
                if (bcast) { if (full) st4<false>(xrow, mean); else st4_masked(xrow, mean, e0, lo, hi); }
                if (avg_m) {
                    float *mrow = a.m + (int64_t)k * a.ld + e0;
                    if (full) st4<false>(mrow, mmean); else st4_masked(mrow, mmean, e0, lo, hi);
                }
            }
            if (grad) {
                f4 gr = gradient(gd, mean);
                if (!full) gr = mask4(gr, e0, lo, hi);
                gn = square_sum(gr);
            }
        }
    }
    if (!measure) return;
    const Pair total = block_sum2<1>(acc, gn);
    if (threadIdx.x == 0) {
        p.partials[2 * ti] = total.a;
        p.partials[2 * ti + 1] = total.b;
    }
}

// ---------------------------------------------------------------- reduction

// The step that the launch's slot-th measurement followed, and whether a sync
// did too: every step in turn when all are measured, else the syncs' steps.
// False if the launch has no such measurement.
__device__ __forceinline__ bool slot_step(const ReduceParams &r, const SpanPlan &sp, int slot, int *j, bool *due) {
    if (r.when.measure) {
        *j = slot;
        *due = slot < sp.n && ((sp.syncs >> slot) & 1);
        return slot < sp.n;
    }
    uint64_t left = sp.syncs;
    for (int i = 0; i < slot; ++i) left &= left - 1;
    *due = left != 0;
    *j = left ? __ffsll((unsigned long long)left) - 1 : 0;
    return left != 0;
}

__device__ __forceinline__ SlotHdr *slot_hdr(const ReduceParams &r, int slot) {
    int i = r.slot0 + slot;   // (a launch has no more slots than the ring)
    if (i >= r.ring) i -= r.ring;
    return reinterpret_cast<SlotHdr *>(r.recs + (int64_t)i * r.slot_bytes);
}

__device__ __forceinline__ void write_hdr(SlotHdr *to, int64_t t, int32_t n, bool due, int32_t p, int32_t p_next,
                                          int32_t status, double S, double GN, double C2, int64_t nC2) {
    SlotHdr h;
    h.t = t;
    h.due = due ? 1 : 0;
    h.p = p;
    h.p_next = p_next;
    h.status = status;
    h.S = S;
    h.GN = GN;
    h.C2 = C2;
    h.nC2 = nC2;
    h.n = n;
    h.pad_ = 0;
    *to = h;
}

// Algorithm 2's sampling and period decision for one measurement (the same
// apply_sync as the host controller), and its record.
__device__ __forceinline__ void control_slot(const ReduceParams &r, const SpanPlan &sp, int slot, int j, bool due,
                                             double S, double GN, SchedState *st) {
    const int64_t t = sp.t + j;
    const int32_t p_t = period_at(r.rule, st->p, t);
    int32_t status = ADPSGD_OK;
    if (due) {
        st->p = p_t;
        // a non-finite S restarts the counter and moves nothing else
        if (!apply_sync(r.rule, t, r.gamma[t - r.when.t], S, st, nullptr)) status = ADPSGD_ENONFINITE;
    }
    write_hdr(slot_hdr(r, slot), t, sp.n, due, p_t, due ? st->p : p_t, status, S, GN, st->C2, st->nC2);
}

// The controller state after the span: t, and the steps since its last sync.
__device__ __forceinline__ void end_span(const ReduceParams &r, const SpanPlan &sp, SchedState *st) {
    const int64_t since = sp.syncs ? sp.n - (64 - __clzll((long long)sp.syncs)) : st->cnt + (sp.t - st->t) + sp.n;
    st->cnt = since;
    st->t = sp.t + sp.n;
}

// Level 1, one wave per chunk (kChunksPerBlock chunks per block), blockIdx.y the
// slot: the chunk's tile partials, summed in a fixed order (strided over the
// lanes, then a butterfly).  A chunk holds at most kChunkTiles = 1024 tiles, 16
// per lane; problems of thousands of small tensors have as many one-tile
// chunks, which would otherwise cost a block each.
constexpr int kChunksPerBlock = kBlock / 64;
__global__ void __launch_bounds__(kBlock) k_reduce_chunks(ReduceParams r) {
    const int slot = blockIdx.y;
    int j;
    bool due;
    if (!slot_step(r, span_plan(r.when, r.sched, r.rule), slot, &j, &due)) return;
    const int lane = threadIdx.x & 63;
    const int64_t ci = ((int64_t)r.block0 + blockIdx.x) * kChunksPerBlock + (threadIdx.x >> 6);
    if (ci >= r.n_chunks) return;  // whole waves: no block-wide barrier follows
    const double *tp = r.tile_partials + slot * r.tile_stride;
    const Chunk c = r.chunks[ci];
    double a = 0.0, b = 0.0;
    if (c.count <= 64) {  // uniform over the wave: one tile partial per lane at most
        if (lane < c.count) {
            a = tp[2 * (int64_t)(c.first + lane)];
            b = tp[2 * (int64_t)(c.first + lane) + 1];
        }
    } else {
        // all of a lane's loads are issued before the first add; the sum is
        // then taken in lane-stride order (the zeros of lanes past the chunk
        // leave it unchanged, so both branches give the same bits)
        constexpr int kPerLane = kChunkTiles / 64;
        static_assert(kPerLane * 64 == kChunkTiles, "chunk tiles per lane");
        double va[kPerLane], vb[kPerLane];
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            const int32_t k = lane + 64 * i;
            const bool in_chunk = k < c.count;
            va[i] = in_chunk ? tp[2 * (int64_t)(c.first + k)] : 0.0;
            vb[i] = in_chunk ? tp[2 * (int64_t)(c.first + k) + 1] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            a += va[i];
            b += vb[i];
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    if (lane == 0) {
        r.chunk_partials[slot * r.chunk_stride + 2 * ci] = a;
        r.chunk_partials[slot * r.chunk_stride + 2 * ci + 1] = b;
    }
}

constexpr int kFinishThreads = 256;
constexpr int kFinishTensors = 512;   // tensors whose sums the finishing block keeps in LDS
// Slots that one finishing block takes in turn, decisions and all: a launch less than a
// block for each and k_control.  A traced adaptive run at p = 1 reserves up to four a
// launch and mostly fills one: 140 steps, K = 4, P = 65,536 2.37 ms with k_control, 1.97
// so; at p = 4, where most are filled, 0.88 and 0.89.
constexpr unsigned kSerialSlots = 4;

// Level 2 for problems with more chunk partials than one LDS window: one block
// per window of tensors (blockIdx.x) and slot (blockIdx.y).  A window of small
// tensors loads its chunk partials (at most kFinishWindow) into LDS and gives
// each tensor to a thread, which adds its chunks in a fixed order (four
// interleaved partial sums); a window holding one large tensor adds its chunks
// strided over the block.  Writes out[tau] = variance (deviation sum / K) and
// out[T + tau] = gradient norm^2 for its tensors, and the window's sums in a
// fixed order to win_partials.
__global__ void __launch_bounds__(kFinishThreads) k_reduce_windows(ReduceParams r) {
    __shared__ double la[kFinishWindow], lb[kFinishWindow];
    const int slot = blockIdx.y;
    int j;
    bool due;
    if (!slot_step(r, span_plan(r.when, r.sched, r.rule), slot, &j, &due)) return;
    const double *cp = r.chunk_partials + slot * r.chunk_stride;
    double *wp = r.win_partials + (int64_t)slot * 2 * r.n_windows;
    double *out = reinterpret_cast<double *>(reinterpret_cast<char *>(slot_hdr(r, slot)) + kSlotHdrBytes);
    const int32_t w = blockIdx.x;
    const int32_t t0 = r.win_begin[w], t1 = r.win_begin[w + 1];
    const int32_t c0 = r.chunk_begin[t0], c1 = r.chunk_begin[t1];
    if (t1 == t0 + 1 && c1 - c0 > kSmallTensorChunks) {  // one large tensor
        double a = 0.0, g = 0.0;
        for (int32_t i = c0 + (int32_t)threadIdx.x; i < c1; i += kFinishThreads) {
            a += cp[2 * (int64_t)i];
            g += cp[2 * (int64_t)i + 1];
        }
        const Pair tot = block_sum2<kFinishThreads / 64>(a, g);
        if (threadIdx.x == 0) {
            const double v = tot.a / (double)r.K;
            out[t0] = v;
            out[r.T + t0] = tot.b;
            wp[2 * w] = v;
            wp[2 * w + 1] = tot.b;
        }
        return;
    }
    const int32_t n = c1 - c0;  // <= kFinishWindow (the host cut the window so)
    for (int32_t i = (int32_t)threadIdx.x; i < n; i += kFinishThreads) {
        la[i] = cp[2 * (int64_t)(c0 + i)];
        lb[i] = cp[2 * (int64_t)(c0 + i) + 1];
    }
    __syncthreads();
    double sa = 0.0, sb = 0.0;
    for (int32_t tau = t0 + (int32_t)threadIdx.x; tau < t1; tau += kFinishThreads) {
        const int32_t b = r.chunk_begin[tau] - c0, e = r.chunk_begin[tau + 1] - c0;
        double a[4] = {0.0, 0.0, 0.0, 0.0}, g[4] = {0.0, 0.0, 0.0, 0.0};
        int32_t i = b;
        for (; i + 4 <= e; i += 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a[q] += la[i + q];
                g[q] += lb[i + q];
            }
        }
        if (i < e) { a[0] += la[i]; g[0] += lb[i]; }
        if (i + 1 < e) { a[1] += la[i + 1]; g[1] += lb[i + 1]; }
        if (i + 2 < e) { a[2] += la[i + 2]; g[2] += lb[i + 2]; }
        const double v = e > b ? ((a[0] + a[1]) + (a[2] + a[3])) / (double)r.K : 0.0;
        const double gn = e > b ? (g[0] + g[1]) + (g[2] + g[3]) : 0.0;
        out[tau] = v;
        out[r.T + tau] = gn;
        sa += v;
        sb += gn;
    }
    const Pair tot = block_sum2<kFinishThreads / 64>(sa, sb);
    if (threadIdx.x == 0) {
        wp[2 * w] = tot.a;
        wp[2 * w + 1] = tot.b;
    }
}

// Level 2 and the decision, one block per slot, or one for all slots in turn.  With at
// most kFinishWindow chunk partials (n_windows = 0) it sums the tensors itself, in a
// fixed order chosen by the tensor's chunk count: a tensor of at most kSmallTensorChunks
// chunks is owned by one thread, which adds its chunks from LDS (four
// interleaved partial sums); a larger tensor is owned by one wave, whose lanes
// add strided chunks from LDS before a butterfly; then out[tau] = variance
// (deviation sum / K), out[T + tau] = gradient norm^2, and S and the norm total
// are block sums.  Otherwise k_reduce_windows has written out, and S and the
// norm total are block sums of its window partials.  With a controller on the
// device a single block's thread 0 then takes Algorithm 2's decisions in step order;
// several blocks leave the sums to k_control, which does.  With none it writes the
// record itself, nothing of which moves at a sync.  out and the record header are
// the host's pinned record slot, written directly.
template <bool ALL>   // one block for all slots
__global__ void __launch_bounds__(kFinishThreads) k_reduce_finish(ReduceParams r) {
    __shared__ double la[kFinishWindow], lb[kFinishWindow];
    __shared__ double lacc[2 * kFinishTensors];   // per-tensor sums, where they fit
    fetch_args<offsetof(ReduceParams, gamma)>();
    const bool decide = r.control && (ALL || r.n_slots == 1);
    auto load_partials = [&](int slot) {
        if (r.n_windows > 0) return;
        // every chunk partial fits one LDS window (the host cuts the tensors into
        // windows for k_reduce_windows otherwise)
        const double *cp = r.chunk_partials + slot * r.chunk_stride;
        for (int32_t i = (int32_t)threadIdx.x; i < r.n_chunks; i += kFinishThreads) {
            la[i] = cp[2 * (int64_t)i];
            lb[i] = cp[2 * (int64_t)i + 1];
        }
    };
    // (the loads are under way while the plan is worked out; of a slot without a
    // measurement they are not used)
    load_partials(blockIdx.x);
    const SpanPlan sp = span_plan(r.when, r.sched, r.rule);
    SchedState st{};   // (thread 0's)
    int slot = blockIdx.x, j;
    bool due;
    for (; slot < r.n_slots && slot_step(r, sp, slot, &j, &due); ++slot) {
        if (ALL && slot > 0) {
            __syncthreads();   // la, lb and lacc of the slot before are read
            load_partials(slot);
        }
        double *out = reinterpret_cast<double *>(reinterpret_cast<char *>(slot_hdr(r, slot)) + kSlotHdrBytes);
        double sa = 0.0, sb = 0.0;
        if (r.n_windows > 0) {
            // the tensors were reduced by k_reduce_windows: add the window sums
            const double *wp = r.win_partials + (int64_t)slot * 2 * r.n_windows;
            for (int32_t w = (int32_t)threadIdx.x; w < r.n_windows; w += kFinishThreads) {
                sa += wp[2 * w];
                sb += wp[2 * w + 1];
            }
        } else {
            double *acc = r.T <= kFinishTensors ? lacc : r.acc + (int64_t)slot * 2 * r.T;
            __syncthreads();   // la, lb
            // small tensors: a thread each
            for (int32_t tau = (int32_t)threadIdx.x; tau < r.T; tau += kFinishThreads) {
                const int32_t b = r.chunk_begin[tau], e = r.chunk_begin[tau + 1];
                if (e - b > kSmallTensorChunks || b >= e) continue;
                double a[4] = {0.0, 0.0, 0.0, 0.0}, g[4] = {0.0, 0.0, 0.0, 0.0};
                int32_t i = b;
                for (; i + 4 <= e; i += 4) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        a[q] += la[i + q];
                        g[q] += lb[i + q];
                    }
                }
                if (i < e) { a[0] += la[i]; g[0] += lb[i]; }
                if (i + 1 < e) { a[1] += la[i + 1]; g[1] += lb[i + 1]; }
                if (i + 2 < e) { a[2] += la[i + 2]; g[2] += lb[i + 2]; }
                acc[tau] = (a[0] + a[1]) + (a[2] + a[3]);
                acc[r.T + tau] = (g[0] + g[1]) + (g[2] + g[3]);
            }
            // large tensors (listed by the host): a wave each, strided lanes, then
            // a butterfly
            const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
            for (int32_t k = wave; k < r.n_large; k += kFinishThreads / 64) {
                const int32_t tau = r.large[k];
                const int32_t cb = r.chunk_begin[tau], ce = r.chunk_begin[tau + 1];
                double a = 0.0, g = 0.0;
                for (int32_t i = cb + lane; i < ce; i += 64) {
                    a += la[i];
                    g += lb[i];
                }
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) {
                    a += __shfl_xor(a, off, 64);
                    g += __shfl_xor(g, off, 64);
                }
                if (lane == 0) {
                    acc[tau] = a;
                    acc[r.T + tau] = g;
                }
            }
            __syncthreads();  // acc of the large tensors, for their owner threads below
            for (int32_t tau = (int32_t)threadIdx.x; tau < r.T; tau += kFinishThreads) {
                double v = 0.0, g = 0.0;
                if (r.chunk_begin[tau + 1] > r.chunk_begin[tau]) {
                    v = acc[tau] / (double)r.K;
                    g = acc[r.T + tau];
                }
                out[tau] = v;
                out[r.T + tau] = g;
                sa += v;
                sb += g;
            }
        }
        const Pair tot = block_sum2<kFinishThreads / 64>(sa, sb);
        if (threadIdx.x == 0) {
            if (decide) {
                if (slot == 0) st = *r.sched;
                control_slot(r, sp, slot, j, due, tot.a, tot.b, &st);
            } else if (r.control) {
                r.sums[2 * slot] = tot.a;
                r.sums[2 * slot + 1] = tot.b;
            } else {
                // (no p, C2 or nC2: they are the host's alone here, and a captured launch
                // serves runs from states that differ in them)
                write_hdr(slot_hdr(r, slot), sp.t + j, sp.n, due, 0, 0,
                          __builtin_isfinite(tot.a) ? ADPSGD_OK : ADPSGD_ENONFINITE, tot.a, tot.b, 0.0, 0);
            }
        }
        if (!ALL) break;
    }
    if (!decide) return;
    const bool none = !slot_step(r, sp, 0, &j, &due);   // no measurement
    if (none) __syncthreads();                         // every thread has read the controller state
    if (threadIdx.x == 0) {
        if (none) {
            st = *r.sched;
            write_hdr(slot_hdr(r, 0), sp.t + sp.n - 1, sp.n, false, st.p, st.p, ADPSGD_OK, 0.0, 0.0, st.C2, st.nC2);
        }
        end_span(r, sp, &st);
        *r.sched = st;
    }
}

// The decisions of a launch of more than kSerialSlots measurements, in step order (one
// thread).
__global__ void __launch_bounds__(64) k_control(ReduceParams r) {
    if (threadIdx.x != 0) return;
    SchedState st = *r.sched;
    const SpanPlan sp = span_plan(r.when, r.sched, r.rule);
    int j;
    bool due;
    for (int slot = 0; slot < r.n_slots && slot_step(r, sp, slot, &j, &due); ++slot)
        control_slot(r, sp, slot, j, due, r.sums[2 * slot], r.sums[2 * slot + 1], &st);
    if (!slot_step(r, sp, 0, &j, &due))
        write_hdr(slot_hdr(r, 0), sp.t + sp.n - 1, sp.n, false, st.p, st.p, ADPSGD_OK, 0.0, 0.0, st.C2, st.nC2);
    end_span(r, sp, &st);
    *r.sched = st;
}

// ---------------------------------------------------------------- problem data

__global__ void __launch_bounds__(kBlock) k_init_problem(float *h, float *xs, int64_t P, RoundKeys rk,
                                                         float log_lo, float log_span, int64_t g0) {
    const int64_t g = g0 + (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t e0 = 4 * g;
    if (e0 >= P) return;
    const u4 rh = philox10(u4{(uint32_t)g, 0u, 0u, TAG_CURVATURE}, rk);
    const f4 hv = f4{expf(fmaf(unif24(rh.x), log_span, log_lo)), expf(fmaf(unif24(rh.y), log_span, log_lo)),
                     expf(fmaf(unif24(rh.z), log_span, log_lo)), expf(fmaf(unif24(rh.w), log_span, log_lo))};
    const f4 xv = normals4(philox10(u4{(uint32_t)g, 0u, 0u, TAG_OPTIMUM}, rk));
    st4_masked(h + e0, hv, e0, 0, P);
    st4_masked(xs + e0, xv, e0, 0, P);
}

// Thread = one float4 group of one row: j = k * groups_per_row + g.
template <bool VEC>
__global__ void __launch_bounds__(kBlock) k_zero_rows(float *a, int64_t ld, int64_t P, int64_t groups_per_row,
                                                      int64_t j0, int64_t n) {
    const int64_t j = j0 + (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= n) return;
    const int64_t k = j / groups_per_row, e0 = 4 * (j - k * groups_per_row);
    float *row = a + k * ld + e0;
    if (VEC && e0 + 4 <= P) st4<false>(row, splat(0.0f));
    else st4_masked(row, splat(0.0f), e0, 0, P);
}

// Rows 1 .. K - 1 = row 0; thread = one float4 group of one row (from row 1 on).
template <bool VEC>
__global__ void __launch_bounds__(kBlock) k_spread_row(float *a, int64_t ld, int64_t P, int64_t groups_per_row,
                                                       int64_t j0, int64_t n) {
    const int64_t j = j0 + (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= n) return;
    const int64_t k = j / groups_per_row, e0 = 4 * (j - k * groups_per_row);
    float *row = a + (k + 1) * ld + e0;
    if (VEC && e0 + 4 <= P) st4<false>(row, ld4<false>(a + e0));
    else st4_masked(row, ld4_masked(a + e0, e0, 0, P), e0, 0, P);
}

// The words of counter (g, c1, c2, c3) as the kernels form them: the noise's (tag 0)
// as a step does, those of the problem data (and of any other tag) as k_init_problem.
__device__ __forceinline__ u4 dump_words(const RoundKeys &rk, uint32_t g, uint32_t c1, uint32_t c2, uint32_t c3) {
    if (c3 == TAG_NOISE) return philox_noise(philox_group(g, rk), c1, c2, rk, noise_keys<8>(rk));
    return philox10(u4{g, c1, c2, c3}, rk);
}

__global__ void __launch_bounds__(kBlock) k_philox_dump(RoundKeys rk, uint32_t c1, uint32_t c2, uint32_t c3,
                                                        int64_t g0, int64_t n, uint32_t *out) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= n) return;
    *reinterpret_cast<u4 *>(out + 4 * j) = dump_words(rk, (uint32_t)(g0 + j), c1, c2, c3);
}

__global__ void __launch_bounds__(kBlock) k_normal_dump(RoundKeys rk, uint32_t c1, uint32_t c2, uint32_t c3,
                                                        int64_t g0, int64_t n, float *out) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= n) return;
    const u4 r = dump_words(rk, (uint32_t)(g0 + j), c1, c2, c3);
    constexpr float kSqrt2Ln2 = 1.17741002251547469101f;   // a step's scale with sigma = 1
    *reinterpret_cast<f4 *>(out + 4 * j) = c3 == TAG_NOISE ? add_noise4(kSqrt2Ln2, r, splat(0.0f)) : normals4(r);
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Blocks of `threads` work-items that one launch may hold (a multiple of 8).
constexpr int64_t piece_blocks(int threads) { return (kMaxLaunchItems / threads) & ~int64_t(7); }

// launch(first block, block count) over [0, n_blocks) in pieces of at most
// piece_blocks(threads) blocks.
template <class F>
hipError_t in_pieces(int64_t n_blocks, int threads, F launch) {
    const int64_t step = piece_blocks(threads);
    for (int64_t b0 = 0; b0 < n_blocks; b0 += step) {
        launch(b0, (unsigned)std::min(step, n_blocks - b0));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The same for the element-wise kernels: launch(first group, group count) in
// pieces of whole blocks of kBlock groups.
template <class F>
hipError_t groups_in_pieces(int64_t n, F launch) {
    const int64_t step = piece_blocks(kBlock) * kBlock;
    for (int64_t g0 = 0; g0 < n; g0 += step) {
        const int64_t m = std::min(step, n - g0);
        launch(g0, m, blocks_for(m));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Dynamic LDS that holds a CU to `cap` resident blocks of a kernel with
// static_lds bytes of its own: each block then takes kLdsPerCU / cap bytes
// (rounded down to 512).  0 for no cap, or when the kernel's own LDS already
// allows no more.
inline int cap_lds(int cap, size_t static_lds) {
    if (cap <= 0) return 0;
    const size_t per_block = (size_t)(kLdsPerCU / cap) & ~size_t(511);
    return per_block > static_lds ? (int)(per_block - static_lds) : 0;
}

template <class Kern>
size_t static_lds_of(Kern kern) {
    hipFuncAttributes fa;
    return hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(kern)) == hipSuccess ? fa.sharedSizeBytes : 0;
}

// Does the K-argument sync kernel take K (else the loop kernel does)?  Two rows
// per wave up to K = 32, four up to 64 and eight up to 128 (the last wave of a
// K that is not a multiple holds fewer): a CU holds at most two blocks of 9-16
// waves, and several rows per wave keep more bytes in flight.  K = 3 is the
// exception: one row per wave in a span, and the loop kernel for the separate
// sync (76% of peak, against 58% and 48% for three one-row or two two-row
// waves); both add the rows in row order, so the replicas keep the same bits.
constexpr bool any_k_kernel(int K, bool average) {
    if (K == 3) return !average;
    return K > 0 && K <= kMaxRegisterK;
}
constexpr int any_k_rows(int K) { return K == 3 ? 1 : (K <= 32 ? 2 : (K <= 64 ? 4 : 8)); }
constexpr int any_k_waves(int K) { return (K + any_k_rows(K) - 1) / any_k_rows(K); }

template <int KT, bool VEC, bool NT, bool AVGM, int RD, bool RAGGED>
hipError_t average_variant(const SyncParams &p, int cap, hipStream_t st) {
    const int threads = KT > 0 ? 64 * average_waves<KT>() : 64 * any_k_waves(p.s.K);
    int lds = 0;
    if (cap > 0) {   // (the attribute query only when it is needed: not under graph capture)
        static const size_t own = static_lds_of(k_average<KT, VEC, NT, AVGM, RD, RAGGED>);
        lds = cap_lds(cap, own);
    }
    return in_pieces(p.n_chunks, threads, [&](int64_t b0, unsigned nb) {   // a block per chunk
        SyncParams q = p;
        q.s.block0 = b0;
        k_average<KT, VEC, NT, AVGM, RD, RAGGED><<<dim3(nb), dim3(threads), lds, st>>>(q);
    });
}

template <int KT, int RD = 0, bool RAGGED = false>
hipError_t average_dispatch(const SyncParams &p, bool avg_m, bool vec, bool nt, int cap, hipStream_t st) {
    if (avg_m) {
        if (vec && nt) return average_variant<KT, true, true, true, RD, RAGGED>(p, cap, st);
        if (vec) return average_variant<KT, true, false, true, RD, RAGGED>(p, cap, st);
        return average_variant<KT, false, false, true, RD, RAGGED>(p, cap, st);
    }
    if (vec && nt) return average_variant<KT, true, true, false, RD, RAGGED>(p, cap, st);
    if (vec) return average_variant<KT, true, false, false, RD, RAGGED>(p, cap, st);
    return average_variant<KT, false, false, false, RD, RAGGED>(p, cap, st);
}

// Dynamic LDS of a k_span block of `waves` waves with K an argument: part and dev.
constexpr int span_lds(int waves) { return waves * 64 * (int)(sizeof(f4) + sizeof(double)); }

template <int KT, int R, bool FEW = false>
hipError_t span_variant(const SpanParams &p, bool vec, bool nt, hipStream_t st) {
    const int threads = KT > 0 ? 64 * span_waves<KT, R, FEW>() : 64 * any_k_waves(p.s.K);
    const int lds = KT > 0 ? 0 : span_lds(any_k_waves(p.s.K));
    return in_pieces(p.n_chunks, threads, [&](int64_t b0, unsigned nb) {   // a block per chunk
        SpanParams q = p;
        q.s.block0 = b0;
        if (vec && nt) k_span<KT, R, true, true, FEW><<<dim3(nb), dim3(threads), lds, st>>>(q);
        else if (vec) k_span<KT, R, true, false, FEW><<<dim3(nb), dim3(threads), lds, st>>>(q);
        else k_span<KT, R, false, false, FEW><<<dim3(nb), dim3(threads), lds, st>>>(q);
    });
}

// A compiled K runs a span in one of three layouts.  One row per wave (two at K =
// 32) streams best and has the most waves: launches of one and two steps, bound by HBM
// (K = 8, P = 11.2M, single steps with their sync 1.08 ms for four against 1.13 with
// eight rows per wave).  What counts is the most steps that the launch may take: one
// that the device ends, with an adaptive period of 1 or 2, may take 3 to 5 and has more
// rows per wave, although it mostly ends sooner.  More rows per wave share the lanes' Philox products and the
// work of a sync, and with all rows in one wave a sync needs no barrier: 32 steps at
// K = 8, P = 138M 22.3 ms with two rows per wave, 20.6 with eight; 60 steps at K =
// 4, P = 20M 3.70 (two) and 3.44 (four); 400 at K = 32, P = 1.2M 10.1-11.1 (four)
// and 9.1 (eight); but 100 at K = 16, P = 25.6M 22.0 (four) and 22.5 (eight; 22.7 in
// one wave of 16 rows, which leaves two waves a SIMD).  A layout needs two waves
// for every SIMD: 64 steps with 8 syncs at K = 4, P = 65,536 take 19 us in 1024
// one-row waves, 29 in 512 of two.
template <int KT, int WIDE, int MID, int TALL>
hipError_t span_dispatch(const SpanParams &p, bool vec, bool nt, hipStream_t st) {
    auto fills = [&](int waves) { return p.n_chunks * waves >= 2 * kSimds; };
    if (p.when.n >= 3 || KT == 32) {
        if (fills(span_waves<KT, TALL, false>())) return span_variant<KT, TALL>(p, vec, nt, st);
        if (fills(span_waves<KT, MID, false>())) return span_variant<KT, MID>(p, vec, nt, st);
    }
    return span_variant<KT, WIDE>(p, vec, nt, st);
}

template <bool STEP>
hipError_t loop_variant(const SpanParams &p, int64_t n_tiles, bool vec, hipStream_t st) {
    return in_pieces(n_tiles, 64, [&](int64_t b0, unsigned nb) {
        SpanParams q = p;
        q.s.block0 = b0;
        if (vec) k_sync_loop<true, STEP><<<dim3(nb), dim3(64), 0, st>>>(q);
        else k_sync_loop<false, STEP><<<dim3(nb), dim3(64), 0, st>>>(q);
    });
}

}  // namespace

int64_t local_step_blocks(int64_t n_groups, int32_t K, const StepShape &shape) {
    const int64_t chunks = (n_groups + shape.block - 1) / shape.block;
    const int64_t per = 8 * (int64_t)shape.row_chunks;  // chunks of one super-chunk
    return ((chunks + per - 1) / per) * per * (int64_t)K;
}

template <int BS>
hipError_t local_step_bs(const StepParams &p, bool vec, bool nt, const StepShape &shape, hipStream_t st) {
    // shape.lds: dynamic LDS per block that the kernel never touches (an occupancy cap)
    const int lds = p.n < kUncappedSteps ? shape.lds : 0;
    return in_pieces(local_step_blocks(p.n_groups, p.K, shape), BS, [&](int64_t b0, unsigned nb) {
        StepParams q = p;
        q.row_chunks = shape.row_chunks;
        q.block0 = b0;
        const bool tail = (p.P & 3) != 0;
        if (vec && nt && tail) k_local_step<BS, true, true, true><<<dim3(nb), dim3(BS), lds, st>>>(q);
        else if (vec && nt) k_local_step<BS, true, true, false><<<dim3(nb), dim3(BS), lds, st>>>(q);
        else if (vec && tail) k_local_step<BS, true, false, true><<<dim3(nb), dim3(BS), lds, st>>>(q);
        else if (vec) k_local_step<BS, true, false, false><<<dim3(nb), dim3(BS), lds, st>>>(q);
        else k_local_step<BS, false, false, false><<<dim3(nb), dim3(BS), lds, st>>>(q);
    });
}

hipError_t launch_local_step(const StepParams &p, bool vec, bool nt, const StepShape &shape, hipStream_t st) {
    if (shape.lds < 0 || shape.lds > kMaxStepLds) return hipErrorInvalidValue;
    if (shape.row_chunks < 1 || shape.row_chunks > kMaxRowChunks) return hipErrorInvalidValue;
    if (p.n < 1 || p.n > kSpanSteps) return hipErrorInvalidValue;
    if (p.n_groups <= 0) return hipSuccess;
    switch (shape.block) {
    case 64: return local_step_bs<64>(p, vec, nt, shape, st);
    case 128: return local_step_bs<128>(p, vec, nt, shape, st);
    case 256: return local_step_bs<256>(p, vec, nt, shape, st);
    default: return hipErrorInvalidValue;
    }
}

int average_tile_waves(int K) {
    switch (K) {
    case 1: return average_waves<1>();
    case 2: return average_waves<2>();
    case 4: return average_waves<4>();
    case 8: return average_waves<8>();
    case 16: return average_waves<16>();
    case 32: return average_waves<32>();
    default: return any_k_kernel(K, true) ? any_k_waves(K) : 0;
    }
}

hipError_t launch_average(const SyncParams &p, int64_t n_tiles, bool avg_m, bool vec, bool nt, int cap,
                          hipStream_t st) {
    if (n_tiles <= 0) return hipSuccess;
    const int K = p.s.K;
    switch (K) {
    case 1: return average_dispatch<1>(p, avg_m, vec, nt, cap, st);
    case 2: return average_dispatch<2>(p, avg_m, vec, nt, cap, st);
    case 4: return average_dispatch<4>(p, avg_m, vec, nt, cap, st);
    case 8: return average_dispatch<8>(p, avg_m, vec, nt, cap, st);
    case 16: return average_dispatch<16>(p, avg_m, vec, nt, cap, st);
    case 32: return average_dispatch<32>(p, avg_m, vec, nt, cap, st);
    default: break;
    }
    if (!any_k_kernel(K, true)) {
        SpanParams q{};
        static_cast<SyncParams &>(q) = p;
        q.avg_m = avg_m ? 1 : 0;
        return loop_variant<false>(q, n_tiles, vec, st);
    }
    switch (any_k_rows(K)) {
    case 2:
        return K % 2 == 0 ? average_dispatch<0, 2, false>(p, avg_m, vec, nt, cap, st)
                          : average_dispatch<0, 2, true>(p, avg_m, vec, nt, cap, st);
    case 4:
        return K % 4 == 0 ? average_dispatch<0, 4, false>(p, avg_m, vec, nt, cap, st)
                          : average_dispatch<0, 4, true>(p, avg_m, vec, nt, cap, st);
    default: return average_dispatch<0, 8, true>(p, avg_m, vec, nt, cap, st);
    }
}

bool span_in_registers(int K) { return K <= kMaxRegisterK; }

hipError_t launch_span(const SpanParams &p, int64_t n_tiles, bool vec, bool nt, bool step_nt, const StepShape &shape,
                       hipStream_t st) {
    if (p.when.n < 1 || p.when.n > kSpanSteps) return hipErrorInvalidValue;
    if (n_tiles <= 0) return hipSuccess;
    const int K = p.s.K;
    switch (K) {
    case 1: return span_variant<1, 1>(p, vec, nt, st);
    case 2: return span_dispatch<2, 1, 2, 2>(p, vec, nt, st);
    case 4: return span_dispatch<4, 1, 2, 4>(p, vec, nt, st);
    case 8: return span_dispatch<8, 1, 2, 8>(p, vec, nt, st);
    case 16: return span_dispatch<16, 1, 4, 4>(p, vec, nt, st);
    case 32: return span_dispatch<32, 2, 4, 8>(p, vec, nt, st);
    default: break;
    }
    if (any_k_kernel(K, false)) {
        const bool few = any_k_waves(K) <= kFewWaves;
        switch (any_k_rows(K)) {
        case 1: return span_variant<0, 1, true>(p, vec, nt, st);
        case 2: return few ? span_variant<0, 2, true>(p, vec, nt, st) : span_variant<0, 2>(p, vec, nt, st);
        case 4: return few ? span_variant<0, 4, true>(p, vec, nt, st) : span_variant<0, 4>(p, vec, nt, st);
        default: return span_variant<0, 8>(p, vec, nt, st);
        }
    }
    // too many workers for the registers: the steps before each measured one in
    // one launch, then that step with the loop kernel (a span that the device
    // ends is one step here)
    if (p.when.device) return p.when.n == 1 ? loop_variant<true>(p, n_tiles, vec, st) : hipErrorInvalidValue;
    int slot = 0;
    for (int j = 0; j < p.when.n;) {
        int to = j;
        while (to < p.when.n && !p.when.measure && !((p.when.syncs >> to) & 1)) ++to;
        SpanParams q = p;
        auto from = [&](int first, int n) {   // q's steps: first .. first + n - 1 of the span
            q.s.t = p.s.t + (uint32_t)first;
            q.s.n = n;
            std::copy(p.s.gamma + first, p.s.gamma + first + n, q.s.gamma);
        };
        if (to > j) {
            from(j, to - j);
            if (const hipError_t e = launch_local_step(q.s, vec, step_nt, shape, st)) return e;
        }
        if (to < p.when.n) {
            from(to, 1);
            q.when.t = p.when.t + to;
            q.when.n = 1;
            q.when.syncs = (p.when.syncs >> to) & 1;
            q.partials = p.partials + (int64_t)slot++ * p.slot_stride;
            if (const hipError_t e = loop_variant<true>(q, n_tiles, vec, st)) return e;
        }
        j = to + 1;
    }
    return hipSuccess;
}

bool chunk_segments(const std::vector<Tile> &tiles, int64_t n_chunks, std::vector<int32_t> *out) {
    out->assign((size_t)n_chunks + 1, -1);
    int64_t prev = -1;
    for (size_t sgi = 0; sgi < tiles.size(); ++sgi) {
        const int64_t c = tiles[sgi].start / kTileElems;
        if (c < 0 || c >= n_chunks || c < prev) return false;
        if (c != prev) (*out)[(size_t)c] = (int32_t)sgi;
        prev = c;
    }
    (*out)[(size_t)n_chunks] = (int32_t)tiles.size();
    for (int64_t c = 0; c < n_chunks; ++c)
        if ((*out)[(size_t)c] < 0) return false;
    return true;
}

hipError_t launch_reduce(const ReduceParams &r, hipStream_t st) {
    const unsigned slots = (unsigned)r.n_slots;
    if (r.n_chunks > 0 && !r.chunks_are_tiles) {
        const int64_t blocks = (r.n_chunks + kChunksPerBlock - 1) / kChunksPerBlock;
        const hipError_t e = in_pieces(blocks, kBlock, [&](int64_t b0, unsigned nb) {
            ReduceParams q = r;
            q.block0 = (int32_t)b0;
            k_reduce_chunks<<<dim3(nb, slots), dim3(kBlock), 0, st>>>(q);
        });
        if (e != hipSuccess) return e;
    }
    if (r.n_windows > 0) {
        k_reduce_windows<<<dim3((unsigned)r.n_windows, slots), dim3(kFinishThreads), 0, st>>>(r);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const bool all = r.control && slots > 1 && slots <= kSerialSlots;
    if (all) k_reduce_finish<true><<<dim3(1), dim3(kFinishThreads), 0, st>>>(r);
    else k_reduce_finish<false><<<dim3(slots), dim3(kFinishThreads), 0, st>>>(r);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !r.control || all || slots == 1) return e;
    k_control<<<dim3(1), dim3(64), 0, st>>>(r);
    return hipGetLastError();
}

hipError_t launch_init_problem(float *h, float *xs, int64_t P, uint64_t seed, double h_lo, double h_hi,
                               hipStream_t st) {
    if (P <= 0) return hipSuccess;
    const double llo = std::log(h_lo), lhi = std::log(h_hi);
    const RoundKeys rk = round_keys(seed);
    return groups_in_pieces((P + 3) / 4, [&](int64_t g0, int64_t, unsigned nb) {
        k_init_problem<<<dim3(nb), dim3(kBlock), 0, st>>>(h, xs, P, rk, (float)llo, (float)(lhi - llo), g0);
    });
}

hipError_t launch_zero_rows(float *a, int64_t ld, int64_t P, int32_t K, bool vec, hipStream_t st) {
    if (P <= 0 || K <= 0) return hipSuccess;
    const int64_t gpr = (P + 3) / 4, n = gpr * K;
    return groups_in_pieces(n, [&](int64_t j0, int64_t, unsigned nb) {
        if (vec) k_zero_rows<true><<<dim3(nb), dim3(kBlock), 0, st>>>(a, ld, P, gpr, j0, n);
        else k_zero_rows<false><<<dim3(nb), dim3(kBlock), 0, st>>>(a, ld, P, gpr, j0, n);
    });
}

hipError_t launch_spread_row(float *a, int64_t ld, int64_t P, int32_t K, bool vec, hipStream_t st) {
    if (P <= 0 || K <= 1) return hipSuccess;
    const int64_t gpr = (P + 3) / 4, n = gpr * (K - 1);
    return groups_in_pieces(n, [&](int64_t j0, int64_t, unsigned nb) {
        if (vec) k_spread_row<true><<<dim3(nb), dim3(kBlock), 0, st>>>(a, ld, P, gpr, j0, n);
        else k_spread_row<false><<<dim3(nb), dim3(kBlock), 0, st>>>(a, ld, P, gpr, j0, n);
    });
}

hipError_t launch_philox_dump(uint64_t seed, uint32_t c1, uint32_t c2, uint32_t c3, int64_t g0, int64_t n,
                              uint32_t *out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const RoundKeys rk = round_keys(seed);
    return groups_in_pieces(n, [&](int64_t j0, int64_t m, unsigned nb) {
        k_philox_dump<<<dim3(nb), dim3(kBlock), 0, st>>>(rk, c1, c2, c3, g0 + j0, m, out + 4 * j0);
    });
}

hipError_t launch_normal_dump(uint64_t seed, uint32_t c1, uint32_t c2, uint32_t c3, int64_t g0, int64_t n,
                              float *out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const RoundKeys rk = round_keys(seed);
    return groups_in_pieces(n, [&](int64_t j0, int64_t m, unsigned nb) {
        k_normal_dump<<<dim3(nb), dim3(kBlock), 0, st>>>(rk, c1, c2, c3, g0 + j0, m, out + 4 * j0);
    });
}

}  // namespace adpsgd
