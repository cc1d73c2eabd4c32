/* Exhaustive CPU check of the step kernel's Box-Muller arithmetic against its definition.
 *
 *  1. Radius: rho = sqrt(-2 ln u), u = (2 (x >> 9) + 1) 2^-24, by the definition's operations
 *     (log by the odd series of 2 atanh, Newton reciprocals and reciprocal square roots), against
 *     the kernel's form, which returns g with rho = -2 g and folds powers of two into constants.
 *     All 2^23 values of x >> 9.
 *  2. The factor -2: sqrt(dN) (rho c) against (-2 sqrt(dN)) (g c), for every g and several c, dN.
 *  3. Quarter-turn parity: bit 30 of y against |y as a float| < 2.  All 2^32 words.
 *  4. e^x scaling: p 2^n by multiplication with the assembled power against ldexp, n = -116 .. 0.
 */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

static float as_f(uint32_t b) { float f; memcpy(&f, &b, 4); return f; }
static uint32_t as_u(float f) { uint32_t b; memcpy(&b, &f, 4); return b; }

static float recip(float x) {
    float y = as_f(0x7EF311C3u - as_u(x));
    for (int i = 0; i < 3; ++i) {
        const float e = fmaf(-x, y, 1.0f);
        y = fmaf(y, e, y);
    }
    return y;
}

static float rho_definition(uint32_t m) {
    const float x = (float)(2 * m + 1) * 0x1p-24f;
    int e;
    float f = frexpf(x, &e);                /* x = f 2^e, f in [1/2, 1) */
    f *= 2.0f;
    e -= 1;
    if (f > 1.41421354f) { f *= 0.5f; e += 1; }
    const float s = (f - 1.0f) * recip(f + 1.0f);
    const float z = s * s;
    float p = 1.0f / 9.0f;
    p = fmaf(p, z, 1.0f / 7.0f);
    p = fmaf(p, z, 1.0f / 5.0f);
    p = fmaf(p, z, 1.0f / 3.0f);
    const float t = s + s;
    const float lf = fmaf(t * z, p, t);
    const float ef = (float)e;
    const float L = fmaf(ef, 0.693145751953125f, fmaf(ef, 1.42860682030941723212e-6f, lf));
    const float q = -2.0f * L;
    float y = as_f(0x5F3759DFu - (as_u(q) >> 1));
    const float h = 0.5f * q;
    for (int i = 0; i < 3; ++i) {
        const float yy = y * y;
        const float d = fmaf(-h, yy, 0.5f);
        y = fmaf(y, d, y);
    }
    return q * y;
}

static float g_kernel(uint32_t m) {
    const uint32_t x = m << 9;
    const float u = as_f((uint32_t)((((uint64_t)0x7Fu << 32) | x) >> 9)) + (0x1p-24f - 1.0f);
    const uint32_t b = as_u(u);
    const int ne = (int32_t)(0x3FB504F3u - b) >> 23;
    const float f = as_f(((uint32_t)ne << 23) + b);
    const float t = fmaf(f, 2.0f, -2.0f) * recip(f + 1.0f);
    const float T = t * t;
    float p = (1.0f / 9.0f) * 0x1p-8f;
    p = fmaf(p, T, (1.0f / 7.0f) * 0x1p-6f);
    p = fmaf(p, T, (1.0f / 5.0f) * 0x1p-4f);
    p = fmaf(p, T, (1.0f / 3.0f) * 0x1p-2f);
    const float lf = fmaf(t * T, p, t);
    const float nf = (float)ne;
    const float L = fmaf(nf, -0.693145751953125f, fmaf(nf, -1.42860682030941723212e-6f, lf));
    float y = as_f(0x9EF759DFu - (as_u(L) >> 1));
    for (int i = 0; i < 3; ++i) {
        const float yy = y * y;
        const float e = fmaf(L, yy, 0.5f);
        y = fmaf(y, e, y);
    }
    return L * y;
}

int main(void) {
    unsigned long long bad_rho = 0, bad_scale = 0, bad_turn = 0, bad_exp = 0;
    static const float cs[4] = {1.0f, 0.70710677f, 3.7450706e-7f, -0.3123f};
    static const float dN[3] = {1e-2f, 5e-4f, 1e-5f};
    for (uint32_t m = 0; m < (1u << 23); ++m) {
        const float rho = rho_definition(m), g = g_kernel(m);
        if (as_u(rho) != as_u(-2.0f * g)) ++bad_rho;
        for (int i = 0; i < 4; ++i)
            for (int j = 0; j < 3; ++j) {
                const float sq = sqrtf(dN[j]);
                const float a = sq * (rho * cs[i]), b = (-2.0f * sq) * (g * cs[i]);
                if (as_u(a) != as_u(b)) ++bad_scale;
            }
    }
    for (uint64_t y = 0; y < (1ull << 32); ++y) {
        const int even = fabsf(as_f((uint32_t)y)) < 2.0f;
        if (even != !((y >> 30) & 1u)) ++bad_turn;
    }
    for (int n = -116; n <= 0; ++n)
        for (uint32_t b = 0x3F330000u; b < 0x3FB60000u; b += 257u) {
            const float p = as_f(b);
            if (as_u(p * as_f((uint32_t)(n + 127) << 23)) != as_u(ldexpf(p, n))) ++bad_exp;
        }
    printf("radius mismatches %llu, scale mismatches %llu, parity mismatches %llu, exp mismatches %llu\n", bad_rho, bad_scale,
           bad_turn, bad_exp);
    return bad_rho || bad_scale || bad_turn || bad_exp;
}
