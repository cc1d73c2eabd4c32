// fpt_device.h -- device-side arithmetic of one Euler-Maruyama step of the
// biased slow-roll Langevin equation, for gfx950.
//
// Method: arXiv:2206.11234, Sec. 2.1-2.3.  Every binary32 operation below is
// part of the step semantics shared with the CPU oracle: the step count of a
// run is decided in binary32, so the order of operations and the places where
// fma is used are fixed (the library is built with -ffp-contract=off and no
// fast-math).  Reciprocals and square roots are fma-only Newton sequences:
// cheaper on gfx950 than the IEEE division/sqrt expansions and reproducible
// operation for operation on any IEEE binary32 machine.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fpt {

enum : int { POT_QUADRATIC = 0, POT_QUADRATIC_BUMP = 1, POT_FLAT = 2 };
enum : int { BIAS_NONE = 0, BIAS_NOISE_SCALED = 1, BIAS_POWER = 2, BIAS_MLP = 3 };
enum : int { ST_RUNNING = 0, ST_ENDED = 1, ST_CENSORED = 2, ST_ESCAPED = 3 };

// ---------------------------------------------------------------------------
// Counter-based noise: Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
// Ten rounds of two 32x32->64 multiplies; the key advances by the Weyl
// constants between rounds.  The key (the seed) is wave-uniform.  One 32x32->64 multiply gives both
// halves of a product (v_mad_u64_u32), and one v_bitop3_b32 (truth table 0x96 = a ^ b ^ c) each
// three-input xor.
// ---------------------------------------------------------------------------
struct U4 {
    uint32_t x, y, z, w;
};

// What the first two Philox rounds of a run's counters (j, t_lo, t_hi, stream) do not share with j:
// round 1's product with t_hi and all of round 2's product with round 1's first word are fixed for
// the run, so they are formed once per run (18 multiplies a call instead of 20, and three two-input
// xors for three-input ones).
struct PhiloxRun {
    uint32_t a;       // stream ^ key1: the second word entering round 2 is hi(M0 j) ^ a
    uint32_t b;       // round 2's first output word is hi(M1 w) ^ b, w that second word
    uint32_t c;       // round 2's third output word is lo(M0 j) ^ c
    uint32_t d;       // round 2's fourth output word
};

__device__ __forceinline__ PhiloxRun philox_run(uint64_t t, uint32_t stream, uint32_t k0, uint32_t k1) {
    const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * static_cast<uint32_t>(t >> 32);
    const uint32_t n0 = static_cast<uint32_t>(pb >> 32) ^ static_cast<uint32_t>(t) ^ k0;
    const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * n0;
    return PhiloxRun{stream ^ k1, static_cast<uint32_t>(pb) ^ (k0 + 0x9E3779B9u),
                     static_cast<uint32_t>(pa >> 32) ^ (k1 + 0xBB67AE85u), static_cast<uint32_t>(pa)};
}

// philox4x32_10(j, t_lo, t_hi, stream, k0, k1) for the run r was formed from, the same words.
__device__ __forceinline__ U4 philox_block(uint32_t j, const PhiloxRun &r, uint32_t k0, uint32_t k1) {
    const uint64_t p1 = static_cast<uint64_t>(0xD2511F53u) * j;
    const uint64_t p2 = static_cast<uint64_t>(0xCD9E8D57u) * (static_cast<uint32_t>(p1 >> 32) ^ r.a);
    uint32_t c0 = static_cast<uint32_t>(p2 >> 32) ^ r.b, c1 = static_cast<uint32_t>(p2);
    uint32_t c2 = static_cast<uint32_t>(p1) ^ r.c, c3 = r.d;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
#pragma unroll
    for (int round = 2; round < 10; ++round) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * c0;
        const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * c2;
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pb >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pa >> 32), c3, k1, 0x96);
        c0 = n0;
        c1 = static_cast<uint32_t>(pb);
        c2 = n2;
        c3 = static_cast<uint32_t>(pa);
    }
    return U4{c0, c1, c2, c3};
}

// 1/x for positive normal x: Newton-Raphson y <- fma(y, fma(-x, y, 1), y), three
// steps from the seed bits(0x7EF311C3 - bits(x)) (relative error < 5.1%); the result
// is within 0.51 ulp.  Division-free: only fma and integer subtract.  The seed negates the
// exponent by subtracting the float's bits from a constant (J. Blinn, "Floating-point
// tricks", IEEE CG&A 17(4), 1997); 0x7EF311C3 is a published tuning of that constant.
__device__ __forceinline__ float recip_f32(float x) {
    float y = __uint_as_float(0x7EF311C3u - __float_as_uint(x));
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float e = __builtin_fmaf(-x, y, 1.0f);
        y = __builtin_fmaf(y, e, y);
    }
    return y;
}

// sqrt x for positive normal x: reciprocal square root by Newton-Raphson
// y <- fma(y, fma(-x/2, y*y, 1/2), y), three steps from bits(0x5F3759DF - (bits(x) >> 1)),
// then x*y; within 2 ulp.  The seed constant is the one of the Quake III Arena source (1999),
// analysed by C. Lomont, "Fast inverse square root" (2003).
__device__ __forceinline__ float sqrt_f32(float x) {
    float y = __uint_as_float(0x5F3759DFu - (__float_as_uint(x) >> 1));
    const float hx = 0.5f * x;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float yy = y * y;
        const float e = __builtin_fmaf(-hx, yy, 0.5f);
        y = __builtin_fmaf(y, e, y);
    }
    return x * y;
}

// The Box-Muller radius of a Philox word x, times -1/2: g with rho = sqrt(-2 ln u) = -2 g for
// u = (2 (x >> 9) + 1) 2^-24, an odd multiple of 2^-24 in (0, 1).
//
// The definition (the oracle's operations): u exact; ln u = e ln2_hi + (e ln2_lo + ln f) for
// u = 2^e f, f in (sqrt(1/2), sqrt 2] (bit patterns (0x3F3504F3, 0x3FB504F3]), ln f = 2 atanh(s),
// s = (f-1)/(f+1), as the odd series to s^9; rho = x y with x = -2 ln u and y the reciprocal square
// root of x from three Newton steps y <- fma(y, fma(-x/2, y*y, 1/2), y) on the seed
// bits(0x5F3759DF - (bits(x) >> 1)) (the seed of the Quake III Arena source (1999), analysed by
// C. Lomont, "Fast inverse square root" (2003)).
//
// The operations below give the same bits with six instructions fewer, as multiplying by a power of
// two commutes with every rounding here (all values are normal numbers):
//   - u is the float of exponent 1.0 and mantissa x >> 9, plus 2^-24 - 1, exact;
//   - -e comes from a subtraction and a shift, and f from adding it to u's exponent field;
//   - t = 2 s from 2 (f-1), T = t t = 4 s^2, and the series' coefficients carry the factors 1/4;
//   - with L = ln u, x/2 = -L, the seed of x in terms of bits(L) is bits(0x9EF759DF - (bits(L) >> 1)),
//     and x y = -2 (L y): the factor -2 goes to the caller's constant.
//
// Two words at a time, one operation of each in turn: a wave's instruction that needs the one before
// it waits 9 cycles, an independent one 5, and the compiler, which takes every operation to be ready
// at once, orders one chain after the other (a group of steps by the count 1840 cycles of a lone wave,
// now 1450; 70 000 runs on the bump, one or two waves per SIMD, 51.8 ms, now 48.1; four waves per SIMD
// hide it).
__device__ __forceinline__ void in_turn(float x, float y) { asm volatile("" ::"v"(x), "v"(y)); }
__device__ __forceinline__ void in_turn(uint32_t x, uint32_t y) { asm volatile("" ::"v"(x), "v"(y)); }

struct Pair {
    float a, b;
};

template <typename F>
__device__ __forceinline__ Pair each(const Pair &x, F f) {
    Pair r{f(x.a), f(x.b)};
    in_turn(r.a, r.b);
    return r;
}
template <typename F>
__device__ __forceinline__ Pair each(const Pair &x, const Pair &y, F f) {
    Pair r{f(x.a, y.a), f(x.b, y.b)};
    in_turn(r.a, r.b);
    return r;
}
template <typename F>
__device__ __forceinline__ Pair each(const Pair &x, const Pair &y, const Pair &z, F f) {
    Pair r{f(x.a, y.a, z.a), f(x.b, y.b, z.b)};
    in_turn(r.a, r.b);
    return r;
}

__device__ __forceinline__ Pair radius_m2(uint32_t xa, uint32_t xb) {
    auto u0 = [](uint32_t x) { return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, x, 9)); };
    const Pair m{u0(xa), u0(xb)};
    const Pair u = each(m, [](float v) { return v + (0x1p-24f - 1.0f); });
    uint32_t na = 0x3FB504F3u - __float_as_uint(u.a), nb = 0x3FB504F3u - __float_as_uint(u.b);
    in_turn(na, nb);
    const Pair nf{static_cast<float>(static_cast<int32_t>(na) >> 23), static_cast<float>(static_cast<int32_t>(nb) >> 23)};
    na &= 0xFF800000u;
    nb &= 0xFF800000u;
    in_turn(na, nb);
    na += __float_as_uint(u.a);
    nb += __float_as_uint(u.b);
    in_turn(na, nb);
    const Pair f{__uint_as_float(na), __uint_as_float(nb)};
    const Pair f2 = each(f, [](float v) { return __builtin_fmaf(v, 2.0f, -2.0f); });
    const Pair d = each(f, [](float v) { return v + 1.0f; });
    // 1/d as recip_f32
    Pair y = each(d, [](float v) { return __uint_as_float(0x7EF311C3u - __float_as_uint(v)); });
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const Pair e = each(d, y, [](float v, float w) { return __builtin_fmaf(-v, w, 1.0f); });
        y = each(y, e, [](float v, float w) { return __builtin_fmaf(v, w, v); });
    }
    const Pair t = each(f2, y, [](float v, float w) { return v * w; });
    const Pair T = each(t, [](float v) { return v * v; });
    Pair p = each(T, [](float v) { return __builtin_fmaf((1.0f / 9.0f) * 0x1p-8f, v, (1.0f / 7.0f) * 0x1p-6f); });
    p = each(p, T, [](float v, float w) { return __builtin_fmaf(v, w, (1.0f / 5.0f) * 0x1p-4f); });
    p = each(p, T, [](float v, float w) { return __builtin_fmaf(v, w, (1.0f / 3.0f) * 0x1p-2f); });
    const Pair tT = each(t, T, [](float v, float w) { return v * w; });
    Pair L = each(tT, p, t, [](float v, float w, float z) { return __builtin_fmaf(v, w, z); });
    L = each(nf, L, [](float v, float w) { return __builtin_fmaf(v, -1.42860682030941723212e-6f, w); });
    L = each(nf, L, [](float v, float w) { return __builtin_fmaf(v, -0.693145751953125f, w); });
    y = each(L, [](float v) { return __uint_as_float(__float_as_uint(v) >> 1); });
    y = each(y, [](float v) { return __uint_as_float(0x9EF759DFu - __float_as_uint(v)); });
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const Pair yy = each(y, [](float v) { return v * v; });
        const Pair e = each(L, yy, [](float v, float w) { return __builtin_fmaf(v, w, 0.5f); });
        y = each(y, e, [](float v, float w) { return __builtin_fmaf(v, w, v); });
    }
    return each(L, y, [](float v, float w) { return v * w; });
}

// cos(2 pi u), sin(2 pi u) for the uniform u = uniform24(x): nearest quarter q = rint(4u),
// r = u - q/4 in [-1/8, 1/8], Taylor polynomials of sin(2 pi r) to r^9 and cos(2 pi r) to r^10
// with coefficients (+-)(2 pi)^n/n!, then a quarter-turn rotation by q.
// q and r come from the bits of x: with y = x + 2^29 (mod 2^32), q = y >> 30 (mod 4) and
// r = (2 a + 1 - 2^21) 2^-24 for a = bits 9..29 of y, formed exactly as
// (0.5 + (2a + 1) 2^-24) - 0.625 -- the same values as the float reduction of u, for every x.
// odd_mask holds 0x3FFFFE (bits 1..21) in a register the compiler cannot see through, so that the
// mask and the exponent go in with one v_and_or_b32.
__device__ __forceinline__ void sincos2pi_bits(uint32_t xa, uint32_t xb, uint32_t odd_mask, Pair &c_out, Pair &s_out) {
    uint32_t ya = xa + 0x20000000u, yb = xb + 0x20000000u;
    in_turn(ya, yb);
    Pair r{__uint_as_float(((ya >> 8) & odd_mask) | 0x3F000001u), __uint_as_float(((yb >> 8) & odd_mask) | 0x3F000001u)};
    in_turn(r.a, r.b);
    r = each(r, [](float v) { return v - 0.625f; });
    const Pair r2 = each(r, [](float v) { return v * v; });
    Pair ps = each(r2, [](float v) { return __builtin_fmaf(42.058693944897653145f, v, -76.7058597530613858416f); });
    Pair pc = each(r2, [](float v) { return __builtin_fmaf(-26.4262567833743974529f, v, 60.2446413718766603627f); });
    ps = each(ps, r2, [](float v, float w) { return __builtin_fmaf(v, w, 81.6052492760750542034f); });
    pc = each(pc, r2, [](float v, float w) { return __builtin_fmaf(v, w, -85.456817206693727736f); });
    ps = each(ps, r2, [](float v, float w) { return __builtin_fmaf(v, w, -41.341702240399760234f); });
    pc = each(pc, r2, [](float v, float w) { return __builtin_fmaf(v, w, 64.939394022668291491f); });
    ps = each(ps, r2, [](float v, float w) { return __builtin_fmaf(v, w, 6.28318530717958647692f); });
    pc = each(pc, r2, [](float v, float w) { return __builtin_fmaf(v, w, -19.7392088021787172377f); });
    const Pair sn = each(ps, r, [](float v, float w) { return v * w; });
    const Pair cs = each(pc, r2, [](float v, float w) { return __builtin_fmaf(v, w, 1.0f); });
    // quarter-turn rotation by q = y >> 30, branch-free: odd q (bit 30 of y: as a float, y's
    // magnitude is not below 2, infinities and NaN patterns included) swaps (cos, sin); cos changes
    // sign for q = 1, 2 (bit 31 of y + 2^30) and sin for q = 2, 3 (bit 31 of y); IEEE negation
    // is the sign bit
    const bool even_a = __builtin_fabsf(__uint_as_float(ya)) < 2.0f, even_b = __builtin_fabsf(__uint_as_float(yb)) < 2.0f;
    Pair c{even_a ? cs.a : sn.a, even_b ? cs.b : sn.b}, s{even_a ? sn.a : cs.a, even_b ? sn.b : cs.b};
    auto turned = [](uint32_t q, float v) {
        return __uint_as_float(__builtin_amdgcn_bitop3_b32(q, __float_as_uint(v), 0x80000000u, 0x6c));
    };
    c_out = Pair{turned(xa + 0x60000000u, c.a), turned(xb + 0x60000000u, c.b)};
    s_out = Pair{turned(ya, s.a), turned(yb, s.b)};
}

// e^x for x <= 0 (x < -80 gives 0): n = rint(x / ln 2), r = x - n ln2 (two-part),
// Taylor series of e^r to r^7, times 2^n (a normal number: n >= -116).
__device__ __forceinline__ float exp_f32(float x) {
    const bool under = x < -80.0f;
    if (under) x = -80.0f;
    const float n = __builtin_rintf(x * 1.44269504088896340736f);
    float r = __builtin_fmaf(-n, 0.693145751953125f, x);
    r = __builtin_fmaf(-n, 1.42860682030941723212e-6f, r);
    float p = 1.0f / 5040.0f;
    p = __builtin_fmaf(p, r, 1.0f / 720.0f);
    p = __builtin_fmaf(p, r, 1.0f / 120.0f);
    p = __builtin_fmaf(p, r, 1.0f / 24.0f);
    p = __builtin_fmaf(p, r, 1.0f / 6.0f);
    p = __builtin_fmaf(p, r, 0.5f);
    p = __builtin_fmaf(p, r, 1.0f);
    p = __builtin_fmaf(p, r, 1.0f);
    const float y = __builtin_ldexpf(p, static_cast<int>(n));
    return under ? 0.0f : y;
}

// Four standard normals for steps 4j .. 4j+3 of a run, times -1/2: Box-Muller on (u0,u1), (u2,u3).
// xi = -2 n with n a member here: sqrt(dN) xi is n times StepConsts::sq_m2, the same bits.
struct F4 {
    float a, b, c, d;
};

// odd_mask: see sincos2pi_bits.
__device__ __forceinline__ uint32_t normals_mask() {
    uint32_t m = 0x3FFFFEu;
    asm volatile("" : "+v"(m));
    return m;
}

__device__ __forceinline__ F4 normals4(uint32_t j, const PhiloxRun &r, uint32_t key0, uint32_t key1, uint32_t odd_mask) {
    // the key schedule is recomputed by scalar adds at each call: left to itself the compiler
    // hoists all round keys into scalar registers and spills them to vector lanes
    asm volatile("" : "+s"(key0), "+s"(key1));
    const U4 x = philox_block(j, r, key0, key1);
    Pair c, s;
    const Pair g = radius_m2(x.x, x.z);
    sincos2pi_bits(x.y, x.w, odd_mask, c, s);
    return F4{g.a * c.a, g.a * s.a, g.b * c.b, g.b * s.b};
}

// ---------------------------------------------------------------------------
// Per-instance binary32 step constants (rounded once on the host from the
// binary64 inputs).
// ---------------------------------------------------------------------------
struct StepConsts {
    float dN, sq_m2, hdN, cm;     // dN, -2 sqrt dN, dN/2, m/(2 pi sqrt 6) (flat: S)
    float a, phi0, inv_w2, inv_2w2;
    float A, phi_end, phi_uv, two_uv;
    float phi_esc, phi_in;
    int32_t p;
    uint32_t k_max;
};

// S = sqrt(V/3)/(2 pi) at phi and the whole drift D + B, D = -V'/V (Sec. 2.3), B = r S.  D is
// formed as -2/phi (+ the bump's term): 2/phi is exact in the reciprocal, so fma(-2, 1/phi, B)
// rounds D + B once, as adding -2/phi does.
// FAR (bump potential): phi is so far from the bump that its exponential is 0 (exp_f32's underflow,
// (phi - phi0)^2 / (2 w^2) above 80), so that 1 + a g is 1 and the bump's part of D is 0; near
// receives (phi - phi0)^2, from which the caller tells whether that held.
constexpr float BUMP_FAR = 80.0f;

template <int POT>
struct FieldTerms {
    float S;         // noise amplitude
    float y;         // 1/phi
    float corr;      // bump: its part of D
    float near;      // bump: (phi - phi0)^2
};

template <int POT, bool FAR>
__device__ __forceinline__ FieldTerms<POT> field_terms(const StepConsts &C, float phi) {
    FieldTerms<POT> T;
    T.near = 0.0f;
    if constexpr (POT == POT_QUADRATIC) {
        T.y = recip_f32(phi);
        T.S = C.cm * phi;
    } else if constexpr (POT == POT_QUADRATIC_BUMP) {
        const float dphi = phi - C.phi0;
        const float e2 = dphi * dphi;
        T.near = e2;
        if constexpr (FAR) {
            T.corr = 0.0f;
            T.y = recip_f32(phi);
            T.S = (C.cm * phi) * sqrt_f32(1.0f);
            return T;
        }
        const float x = -(e2 * C.inv_2w2);
        const float g = exp_f32(x);
        const float ag = C.a * g;
        const float one_ag = 1.0f + ag;
        const float num = (dphi * C.inv_w2) * ag;
        T.corr = num * recip_f32(one_ag);
        T.y = recip_f32(phi);
        T.S = (C.cm * phi) * sqrt_f32(one_ag);
    } else {
        T.S = C.cm;
    }
    return T;
}

template <int POT, bool BIASED, bool FAR>
__device__ __forceinline__ float drift(const FieldTerms<POT> &T, float B) {
    if constexpr (POT == POT_QUADRATIC || (POT == POT_QUADRATIC_BUMP && FAR)) {
        return BIASED ? __builtin_fmaf(-2.0f, T.y, B) : -2.0f * T.y;
    } else if constexpr (POT == POT_QUADRATIC_BUMP) {
        const float D = __builtin_fmaf(-2.0f, T.y, T.corr);
        return BIASED ? D + B : D;
    } else {
        return BIASED ? B : 0.0f;
    }
}

// r = B/S in noise units (Sec. 2.3 eq. eq_importance_sampling_amplitude_general
// with f = S, and the power law of Sec. 3.4).  P > 0: the power law's exponent, known at compile time; 0: any.
template <int BIAS, int P>
__device__ __forceinline__ float bias_ratio(const StepConsts &C, float phi, float S) {
    if constexpr (BIAS == BIAS_NOISE_SCALED) {
        return C.A;
    } else if constexpr (BIAS == BIAS_POWER) {
        float pw = 1.0f;
        if constexpr (P > 0) {
            pw = phi;
#pragma unroll
            for (int i = 1; i < P; ++i) pw = pw * phi;
        } else {
            for (int i = 0; i < C.p; ++i) pw = pw * phi;
        }
        return (C.A * pw) * recip_f32(S);
    } else {
        return 0.0f;
    }
}

// Status of a run that has stopped, from where it stopped: the end surface takes precedence
// over the step cap, the cap over escape (Sec. 2.1, Sec. 3).
__device__ __forceinline__ int final_status(const StepConsts &C, float phi, uint32_t k) {
    if (phi <= C.phi_end) return ST_ENDED;
    if (k >= C.k_max) return ST_CENSORED;
    return (phi > C.phi_esc) ? ST_ESCAPED : ST_RUNNING;
}

// One Euler-Maruyama step of the biased Langevin equation (Sec. 2.2 eq. eq_euler_maruyam_modified,
// drift, noise and bias at the pre-step point): the field after it, reflected above phi_UV (Sec.
// 2.1, Sec. 3), and the weight increment dlw = -r (r dN/2 + sqrt(dN) xi) that the caller adds to
// ln w in binary64.  n = -xi/2; r_net is the bias when it comes from the learned network.  Returns
// r and writes sqrt(dN) xi, which the training replay reuses.  WALL: the run has a reflecting wall,
// has none, or either.
enum : int { WALL_NONE = 0, WALL_ALL = 1, WALL_ANY = 2 };

template <int POT, int BIAS, int P = 0, int WALL = WALL_ANY, bool FAR = false>
__device__ __forceinline__ float em_step(const StepConsts &C, float &phi, float n, float r_net, float &dlw, float &sxi,
                                         float *near = nullptr) {
    const FieldTerms<POT> T = field_terms<POT, FAR>(C, phi);
    if (near) *near = T.near;
    float r = 0.0f, drift_dN;
    sxi = C.sq_m2 * n;
    if constexpr (BIAS == BIAS_NONE) {
        drift_dN = drift<POT, false, FAR>(T, 0.0f) * C.dN;
    } else {
        if constexpr (BIAS == BIAS_MLP) r = r_net;
        else r = bias_ratio<BIAS, P>(C, phi, T.S);
        drift_dN = drift<POT, true, FAR>(T, r * T.S) * C.dN;
    }
    // The whole increment (D + B) dN + S sqrt(dN) xi is formed first and rounded onto phi once.
    // Adding the deterministic part to phi on its own would round it to phi's grid every step:
    // at small dN it spans only tens of ulps of phi, and its fraction of an ulp changes so slowly
    // with phi that the rounding error repeats from step to step instead of averaging out.
    const float nphi = phi + __builtin_fmaf(T.S, sxi, drift_dN);
    if constexpr (BIAS != BIAS_NONE) dlw = -(r * __builtin_fmaf(r, C.hdN, sxi));
    else dlw = 0.0f;
    // Reflection x -> 2 phi_UV - x above the wall, as a minimum: 2 phi_UV is exact and rounding
    // is monotone, so fl(2 phi_UV - x) <= phi_UV < x exactly when x > phi_UV (and >= x otherwise);
    // with no wall 2 phi_UV is +inf and the minimum is x.
    phi = WALL == WALL_NONE ? nphi : __builtin_fminf(nphi, C.two_uv - nphi);
    return r;
}

// Whether a run stops after step k at phi: the end surface, the step cap or escape (Sec. 2.1,
// Sec. 3); final_status() names which.
__device__ __forceinline__ bool stops(const StepConsts &C, float phi, uint32_t k) {
    return phi <= C.phi_end || k >= C.k_max || phi > C.phi_esc;
}

// A run between groups of four steps: group j's steps are 4j .. 4j+3.
struct RunState {
    float phi;
    uint32_t j;
    double lw;
};

// Groups a run can take whole before the step cap: it stops in group j when j + 1 >= this.
__device__ __forceinline__ uint32_t cap_groups(uint32_t k_max) { return (k_max >> 2) + ((k_max & 3u) != 0u ? 1u : 0u); }

// Where a run stopped, kept apart from the state of its lane, which steps on unread (the step kernels
// keep it in LDS: in registers it took four copies a group).
struct Stopped {
    float phi;
    uint32_t k;
    double lw;
};

// Four steps from R: the field, ln w and (with H) the noise sum after each, and the smallest `near` of
// the four starting points.
struct Steps4 {
    float p[4], h[4];
    double w[4];
    float near;
};

template <int POT, int BIAS, int P, int WALL, bool FAR>
__device__ __forceinline__ Steps4 steps4(const StepConsts &C, const F4 &z, float r_net, const RunState &R, const float *H) {
    const float n[4] = {z.a, z.b, z.c, z.d};
    Steps4 S;
    float phi = R.phi, near[4];
    double lw = R.lw;
    float sum = H ? *H : 0.0f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        float dlw, sxi;
        const float r = em_step<POT, BIAS, P, WALL, FAR>(C, phi, n[s], r_net, dlw, sxi, &near[s]);
        if constexpr (BIAS != BIAS_NONE) lw += static_cast<double>(dlw);
        if (H) sum = sum + __builtin_fmaf(r, C.dN, sxi);
        S.p[s] = phi;
        S.w[s] = lw;
        S.h[s] = sum;
    }
    S.near = __builtin_fminf(__builtin_fminf(near[0], near[1]), __builtin_fminf(near[2], near[3]));
    return S;
}

// Bump potential: the least (phi - phi0)^2 / (2 w^2) at which a group may be taken without the bump, and
// whether the wave's next one is (group4).  It is infinite, and every group is taken with the bump, where
// a run can get so far from it that (phi - phi0) / w^2 overflows: the bump's term is then infinity times
// 0, and leaving it out would give another field.
struct BumpFar {
    float least;
    bool now = false;
};

// The four steps of every lane's group R.j, all taken without a test between them: the group's
// smallest and largest field and the step cap tell at its end whether a run has stopped inside it,
// and then the first step that stops it is picked from the saved fields and weights into F (what the
// steps past it computed is dropped).  Tests after every step cost 7 of 28 instructions, and the
// branches around them kept the compiler from overlapping one step's arithmetic with the next's
// normals.  `running` has the bits of the lanes whose runs go on; the other lanes compute along, so
// that the whole group is one stretch of code.  Returns the lanes whose runs stopped here and takes
// them out of `running`.  H, where not NULL, gains fma(r, dN, sqrt(dN) xi) of each step taken, in
// step order.
//
// Bump potential: far.now tells whether the wave's runs were all far from the bump in the last group;
// then this one is taken without it (65 instructions a step instead of 108), and again with it if a
// run came near.  The rule is the wave's, as a divergent step would issue both; it pays where the
// wave's runs move together (70 000 runs that all fit the launch: 60.3 ms without
// the rule, 52.6 with it; now 48.1).
template <int POT, int BIAS, int P = 0, int WALL = WALL_ANY>
__device__ __forceinline__ uint64_t group4(const StepConsts &C, uint32_t j_cap, const F4 &z, float r_net, RunState &R,
                                           uint64_t &running, Stopped *F, BumpFar &far, float *H = nullptr) {
    Steps4 S;
    if constexpr (POT == POT_QUADRATIC_BUMP) {
        auto came_near = [&]() { return (__builtin_amdgcn_ballot_w64(!(S.near * C.inv_2w2 > far.least)) & running) != 0; };
        if (far.now) {
            S = steps4<POT, BIAS, P, WALL, true>(C, z, r_net, R, H);
            far.now = !came_near();
        }
        if (!far.now) {
            S = steps4<POT, BIAS, P, WALL, false>(C, z, r_net, R, H);
            far.now = !came_near();
        }
    } else {
        S = steps4<POT, BIAS, P, WALL, false>(C, z, r_net, R, H);
    }
    const float *p = S.p, *h = S.h;
    const double *w = S.w;
    if (H) *H = h[3];
    const float lo = __builtin_fminf(__builtin_fminf(p[0], p[1]), __builtin_fminf(p[2], p[3]));
    const uint32_t j = R.j;
    R.phi = p[3];
    R.lw = w[3];
    R.j = j + 1;
    // (no short circuit: its branches would split the group's arithmetic)
    uint64_t m = __builtin_amdgcn_ballot_w64(lo <= C.phi_end) | __builtin_amdgcn_ballot_w64(j + 1 >= j_cap);
    if constexpr (WALL != WALL_ALL) {              // runs with a wall do not escape
        float hi;       // (the compiler's own maximum first canonicalises each operand)
        asm("v_max3_f32 %0, %1, %2, %3" : "=v"(hi) : "v"(p[0]), "v"(p[1]), "v"(p[2]));
        asm("v_max_f32 %0, %1, %2" : "=v"(hi) : "v"(hi), "v"(p[3]));
        m |= __builtin_amdgcn_ballot_w64(hi > C.phi_esc);
    }
    m &= running;
    if (__builtin_expect(m != 0, 0)) {
        running &= ~m;
        if ((m >> __lane_id()) & 1u) {
            const uint32_t left = C.k_max - 4 * j;     // steps to the cap, >= 1
            int s = 3;
            for (int q = 2; q >= 0; --q)
                if (p[q] <= C.phi_end || p[q] > C.phi_esc || static_cast<uint32_t>(q + 1) >= left) s = q;
            F->phi = s == 0 ? p[0] : s == 1 ? p[1] : s == 2 ? p[2] : p[3];
            F->lw = s == 0 ? w[0] : s == 1 ? w[1] : s == 2 ? w[2] : w[3];
            F->k = 4 * j + 1 + static_cast<uint32_t>(s);
            if (H) *H = s == 0 ? h[0] : s == 1 ? h[1] : s == 2 ? h[2] : h[3];
        }
    }
    return m;
}

}  // namespace fpt
