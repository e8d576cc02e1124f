/* Check of the bracketed step of the BF16-state commit: p' = bf16(RN(p - s)) of
 * s = RN(step_size * RN(m / den)) is taken from the two ends
 *   p - ratio * step_size * (1 -+ 2^-k),  ratio = m * rcp(root * rs_bc2 + eps),
 * whenever both round to the same bf16 word inside the accepted ranges.  For every
 * pair of a hardware root and reciprocal that is at most one bit pattern away from the
 * correctly rounded one, an accepted result must be the exact form's.  Operands: a
 * training shard's, random exponents over the whole binary32 range, and all
 * combinations of edge values.  Argument: k (20 in the kernel).  Prints the numbers of
 * results checked, accepted, accepted in the training shard's part, and wrong. */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static float from_bits(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static uint32_t to_bits(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
static uint16_t bf16(float x) {
    const uint32_t u = to_bits(x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
static uint64_t rng_state;
static uint64_t rng(void) {
    uint64_t z = (rng_state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
static float unit(void) { return (float)(rng() >> 40) * 0x1p-24f; }

static unsigned long long checked, accepted, wrong;
static float bracket;

/* p is p * decay, m and v the new moments */
static void check(float p, float m, float v, float step_size, float rs_bc2, float eps) {
    const float den_exact = sqrtf(v) * rs_bc2 + eps;
    const float ratio_exact = m / den_exact;
    const float s_exact = step_size * ratio_exact;
    const uint16_t want = bf16(p - s_exact);
    const float size_lo = step_size * (1.0f - bracket), size_hi = step_size * (1.0f + bracket);
    for (int d = -1; d <= 1; ++d) {
        const float root = from_bits(to_bits(sqrtf(v)) + (uint32_t)d);
        const float den = fmaf(root, rs_bc2, eps);
        for (int r = -1; r <= 1; ++r) {
            const float ratio = m * from_bits(to_bits(1.0f / den) + (uint32_t)r);
            const uint16_t near = bf16(fmaf(ratio, -size_lo, p)), far = bf16(fmaf(ratio, -size_hi, p));
            const uint16_t p_off = (uint16_t)(near * 2 - 2 * 0x2680), v_off = (uint16_t)(bf16(v) - 0x1000);
            ++checked;
            if (!(step_size >= 0x1p-40f && step_size <= 0x1p40f && eps <= 0x1p100f)) continue;
            if (near != far || p_off >= 2 * (0x4980 - 0x2680) || v_off >= 0x7F80 - 0x1000) continue;
            ++accepted;
            if (near != want) ++wrong;
        }
    }
}

static float any_float(void) { return from_bits((uint32_t)rng()); }
static float log_uniform(int lo, int hi) { return ldexpf(1.0f + unit(), lo + (int)(rng() % (uint64_t)(hi - lo))); }
static float sign(float x) { return (rng() & 1) ? -x : x; }

int main(int argc, char** argv) {
    bracket = ldexpf(1.0f, -(argc > 1 ? atoi(argv[1]) : 20));
    for (long k = 0; k < 4000000; ++k) { /* a training shard */
        const float p = sign(0.04f * unit()), m = sign(3e-4f * unit() * unit()), v = 4e-7f * unit() + 1e-12f;
        check(p, m, v, 3e-4f * (1.0f + 9.0f * unit()), 1.0f + 3.0f * unit(), 1e-8f);
    }
    const unsigned long long usual = accepted;
    for (long k = 0; k < 4000000; ++k) { /* p near s, tiny and huge operands */
        const float v = log_uniform(-100, 127), eps = log_uniform(-149, 110), ss = log_uniform(-45, 45);
        const float m = sign(log_uniform(-149, 127)), rs = log_uniform(0, 13);
        const float s = ss * (m / (sqrtf(v) * rs + eps));
        check((rng() & 1) ? s * (1.0f + ldexpf(unit(), -(int)(rng() % 24))) : sign(log_uniform(-60, 30)), m, v, ss, rs, eps);
    }
    for (long k = 0; k < 2000000; ++k) check(any_float(), any_float(), any_float(), log_uniform(-42, 42), 1.0f, 1e-8f);
    static const uint32_t edge[] = {0x00000000, 0x00000001, 0x007FFFFF, 0x00800000, 0x0F800000, 0x10000000, 0x0FFFFFFF,
                                    0x10007FFF, 0x10008000, 0x26800000, 0x267FFFFF, 0x26808000, 0x3F800000, 0x3F7FFFFF,
                                    0x3F808000, 0x49800000, 0x497F7FFF, 0x497F8000, 0x7F7FFFFF, 0x7F7F8000, 0x7F800000,
                                    0x7F800001, 0x7FC00000, 0x7FFFFFFF};
    static const float sizes[] = {0.0f, 0x1p-149f, 0x1p-40f, 3e-4f, 1.0f, 0x1p40f, 0x1p41f, 3e38f};
    static const float epss[] = {0x1p-149f, 1e-8f, 1.0f, 0x1p100f, 3e38f};
    const int n = (int)(sizeof edge / sizeof edge[0]);
    for (int a = 0; a < 2 * n; ++a)
        for (int b = 0; b < 2 * n; ++b)
            for (int c = 0; c < 2 * n; ++c)
                for (int s = 0; s < 8; ++s)
                    for (int e = 0; e < 5; ++e)
                        check(from_bits(edge[a % n] | (uint32_t)(a / n) << 31), from_bits(edge[b % n] | (uint32_t)(b / n) << 31),
                              from_bits(edge[c % n] | (uint32_t)(c / n) << 31), sizes[s], 1.0f + (float)(a % 3), epss[e]);
    printf("%llu %llu %llu %llu\n", checked, accepted, usual, wrong);
    return wrong == 0 ? 0 : 1;
}
