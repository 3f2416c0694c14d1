// Counter-based noise for the local steps, on the device.
//
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, "Parallel Random Numbers: As Easy
// as 1, 2, 3", SC'11): ten rounds of two 32x32->64 multiplies by fixed odd
// multipliers, with the high halves xored into the other two counter words
// and the round key; the key advances by two Weyl constants per round.  The
// key is the 64-bit seed split into two words; it is uniform across a launch.
// The round keys are in scalar registers, or in vector registers where a kernel has
// some to spare (noise_keys).
//
// Gaussian noise by Box-Muller (1958) on the 24 high bits of each word.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace adpsgd {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

struct RoundKeys {
    uint32_t lo[10];
    uint32_t hi[10];
};

__host__ __device__ inline RoundKeys round_keys(uint64_t seed) {
    RoundKeys rk;
    uint32_t a = (uint32_t)seed, b = (uint32_t)(seed >> 32);
    for (int r = 0; r < 10; ++r) {
        rk.lo[r] = a;
        rk.hi[r] = b;
        a += 0x9E3779B9u;  // Weyl increments of the published key schedule
        b += 0xBB67AE85u;
    }
    return rk;
}

// Counter words (c.x, c.y, c.z, c.w) -> 4 random words.
__device__ __forceinline__ u4 philox10(u4 c, const RoundKeys &rk) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t prod_a = (uint64_t)c.x * 0xD2511F53u;
        const uint64_t prod_b = (uint64_t)c.z * 0xCD9E8D57u;
        const uint32_t y = (uint32_t)prod_b;
        const uint32_t w = (uint32_t)prod_a;
        c.x = (uint32_t)(prod_b >> 32) ^ c.y ^ rk.lo[r];
        c.z = (uint32_t)(prod_a >> 32) ^ c.w ^ rk.hi[r];
        c.y = y;
        c.w = w;
    }
    return c;
}

// v in a vector register.  An instruction of single-precision arithmetic or a
// v_bitop3_b32 issues in 2 cycles a wave when all its operands are vector
// registers or constants, and in 4 with a scalar register among them (measured
// with eight waves a SIMD: 1.1-1.2 ns against 1.7-1.9), so what the steps of a
// launch use again and again is kept in vector registers, uniform as it is.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t v) {
    uint32_t r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
    return r;
}
__device__ __forceinline__ float in_vgpr(float v) { return __uint_as_float(in_vgpr(__float_as_uint(v))); }

// v >> 8 in the three-operand encoding, which issues in 2 cycles; the compiler
// would take the short one, which issues in 4.
__device__ __forceinline__ uint32_t shift_right8(uint32_t v) {
    uint32_t r;
    asm("v_lshrrev_b32_e64 %0, 8, %1" : "=v"(r) : "v"(v));
    return r;
}

// Three-input exclusive or (one v_bitop3_b32).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The noise words of group g: counter (g, k, t, 0).  With k and t uniform over
// the wave, round 0's product of t is a scalar, and so is round 1's product of
// the word it makes; the products of g in round 0 and of the word they make in
// round 1 depend on g alone.  A lane that takes several workers or steps of
// its group therefore forms those two once (philox_group), and every (k, t)
// costs eight rounds of vector products instead of ten.
struct PhiloxGroup {
    uint32_t lo0;        // low word of g's product in round 0
    uint32_t hi1, lo1;   // round 1's product of the word it makes
};
__device__ __forceinline__ PhiloxGroup philox_group(uint32_t g, const RoundKeys &rk) {
    const uint64_t a = (uint64_t)g * 0xD2511F53u;
    const uint32_t z = (uint32_t)(a >> 32) ^ rk.hi[0];
    const uint64_t b = (uint64_t)z * 0xCD9E8D57u;
    return PhiloxGroup{(uint32_t)a, (uint32_t)(b >> 32), (uint32_t)b};
}
// The keys of rounds 2 to 9, the first ROUNDS rounds' in vector registers.
template <int ROUNDS>
struct NoiseKeys {
    uint32_t lo[8], hi[8];
};
template <int ROUNDS>
__device__ __forceinline__ NoiseKeys<ROUNDS> noise_keys(const RoundKeys &rk) {
    NoiseKeys<ROUNDS> nk;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        nk.lo[r] = r < ROUNDS ? in_vgpr(rk.lo[r + 2]) : rk.lo[r + 2];
        nk.hi[r] = r < ROUNDS ? in_vgpr(rk.hi[r + 2]) : rk.hi[r + 2];
    }
    return nk;
}
template <int ROUNDS>
__device__ __forceinline__ u4 philox_noise(const PhiloxGroup &pg, uint32_t k, uint32_t t, const RoundKeys &rk,
                                           const NoiseKeys<ROUNDS> &nk) {
    const uint64_t pt = (uint64_t)t * 0xCD9E8D57u;                   // scalar: round 0
    const uint32_t x = (uint32_t)(pt >> 32) ^ k ^ rk.lo[0];
    const uint64_t px = (uint64_t)x * 0xD2511F53u;                   // scalar: round 1
    u4 c;
    c.x = pg.hi1 ^ ((uint32_t)pt ^ rk.lo[1]);
    c.y = pg.lo1;
    c.z = pg.lo0 ^ ((uint32_t)(px >> 32) ^ rk.hi[1]);
    c.w = (uint32_t)px;
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        const uint64_t prod_a = (uint64_t)c.x * 0xD2511F53u;
        const uint64_t prod_b = (uint64_t)c.z * 0xCD9E8D57u;
        c.x = xor3((uint32_t)(prod_b >> 32), c.y, nk.lo[r - 2]);
        c.z = xor3((uint32_t)(prod_a >> 32), c.w, nk.hi[r - 2]);
        c.y = (uint32_t)prod_b;
        c.w = (uint32_t)prod_a;
    }
    return c;
}

// Two Box-Muller normals from two words: radius sqrt(-2 ln u1) with
// u1 = (hi24(a) + 1) 2^-24 in (0, 1] (never 0, so the log is finite) and angle
// 2 pi u2 with u2 = hi24(b) 2^-24.  Both uniforms are exact in fp32.
// The gfx950 transcendental instructions fit this form directly: v_log_f32 is
// log2 (u1 >= 2^-24, so no denormal inputs), and v_sin_f32 / v_cos_f32 take
// the angle in turns, so sin(2 pi u2) needs no range reduction.  This skips
// the special-case handling of the libm-style wrappers, which this input range
// never needs.
__device__ __forceinline__ void box_muller2(uint32_t a, uint32_t b, float &z0, float &z1) {
    const float u1 = (float)((a >> 8) + 1u) * 0x1p-24f;
    const float u2 = (float)(b >> 8) * 0x1p-24f;
    constexpr float kMinus2Ln2 = -1.38629436111989061883f;   // -2 ln 2
    const float radius = __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(u1));
    z0 = radius * __builtin_amdgcn_cosf(u2);
    z1 = radius * __builtin_amdgcn_sinf(u2);
}

__device__ __forceinline__ f4 normals4(u4 r) {
    float z0, z1, z2, z3;
    box_muller2(r.x, r.y, z0, z1);
    box_muller2(r.z, r.w, z2, z3);
    return f4{z0, z1, z2, z3};
}

// base + sigma z for the two normals z of words a and b, with
// s = sigma sqrt(2 ln 2): sigma times the radius is s sqrt(-log2 u1), so the
// noise level and the logarithm's base cost one product for two normals, and
// the cosine's and the sine's product takes the sum.  The bits of n = hi24(a) are
// also the float n 2^-149 (a denormal, or the first normal binade), so the
// product with 2^125 is n 2^-24 without a conversion, exact, and the fma's sum
// with 2^-24 is too.
__device__ __forceinline__ void add_noise2(float s, uint32_t a, uint32_t b, float base0, float base1, float &d0,
                                           float &d1) {
    const float u1 = fmaf(__uint_as_float(shift_right8(a)), 0x1p125f, 0x1p-24f);
    const float u2 = __uint_as_float(shift_right8(b)) * 0x1p125f;
    const float radius = s * __builtin_amdgcn_sqrtf(-__builtin_amdgcn_logf(u1));
    d0 = fmaf(radius, __builtin_amdgcn_cosf(u2), base0);
    d1 = fmaf(radius, __builtin_amdgcn_sinf(u2), base1);
}
__device__ __forceinline__ f4 add_noise4(float s, u4 r, f4 base) {
    float d0, d1, d2, d3;
    add_noise2(s, r.x, r.y, base.x, base.y, d0, d1);
    add_noise2(s, r.z, r.w, base.z, base.w, d2, d3);
    return f4{d0, d1, d2, d3};
}

// Uniform in [0, 1) from the 24 high bits.
__device__ __forceinline__ float unif24(uint32_t r) { return (float)(r >> 8) * 0x1p-24f; }

// Counter layout: (group g = i/4, worker k, step t, tag).
enum : uint32_t { TAG_NOISE = 0u, TAG_CURVATURE = 1u, TAG_OPTIMUM = 2u };

}  // namespace adpsgd
