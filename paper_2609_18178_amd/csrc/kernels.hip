// kernels.hip -- gfx950 kernels of libpactshard.
//
// One tile kernel serves every mode on binary32 state (commit, commit that
// also zeroes the gradient, state digest, bf16 digest, gradient guard) and a
// twin serves state held in BF16 (commit, state digest).
// Work is cut into tiles that never straddle a segment, and
// each workgroup takes exactly one tile (the hardware dispatcher then keeps
// every CU full and balances the tail by itself; a persistent grid measured
// slower on this pattern).  A full, aligned tile moves, per thread and per
// array, one to four 16-byte vectors with buffer_load/store_dwordx4 (shape_of in
// launch.h), and as many 8-byte ones into the bf16 working copy (dwordx2).  All of
// it is marked non-temporal.  A
// segment's tiles begin at its first element that is aligned in every array
// (up to seven elements in), and a last tile that is not full masks its
// vectors; only the elements before the first and behind the last vector, and
// segments whose arrays are never aligned together, go element by element.
//
// The digest is accumulated per thread in a 64-bit register (wrapping add),
// summed over the workgroup with 64-bit LDS atomics (one word per wave), and
// handed in with two 64-bit atomics per workgroup and result; the workgroup that hands in
// the last share of a result slot writes the slot (see "result slots" below),
// so a call is its tile launches alone.  Without a workspace each workgroup
// adds its share to the result slot itself, which a launch before the tiles
// clears.  Wrapping addition is associative and commutative, so the order in
// which workgroups arrive cannot change the result.
//
// Arithmetic is the library contract in pactshard.h: one IEEE binary32
// rounding per operation, no contraction or reassociation (the translation
// unit is built with -ffp-contract=off and without fast-math), correctly
// rounded sqrt and division, fp32 denormals kept.
#include <algorithm>

#include "launch.h"


// No fused multiply-add anywhere in this file, whatever the command line says.
#pragma clang fp contract(off)

namespace pact {
namespace {

// ---------------------------------------------------------------------------
// digest word hash: splitmix64 generator output for state x
// ---------------------------------------------------------------------------
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kMul1 = 0xBF58476D1CE4E5B9ull;
constexpr uint64_t kMul2 = 0x94D049BB133111EBull;
constexpr uint32_t kTagP = 0, kTagM = 1, kTagV = 2, kTagB = 3;  // array tags (bits 56..63 of the index)

// Low 64 bits of z * C for a constant C = CHI:CLO.  With z = hi:lo,
//   z * C mod 2^64 = lo*CLO + ((hi*CLO + lo*CHI) << 32)
// and only the low 32 bits of the cross term hi*CLO + lo*CHI matter:
//   t     = lo * CHI              v_mul_lo_u32
//   cross = hi * CLO + t          v_mad_u64_u32 (t zero-extended; low half used)
//   prod  = lo * CLO              v_mad_u64_u32 (full 64-bit product)
//   res   = prod + (cross << 32)  v_add_u32 on the high half
// Three VOP3 instructions and one VOP2 add.  On gfx950 a VOP3 instruction
// issues at about half the rate of a VOP2 one, and the hash is most of the
// VALU work of every digesting kernel, so the cheaper add in place of a
// 64-bit shift or a fourth multiply counts.  The compiler's own lowering
// takes four multiply-class instructions plus register moves.  VALU-only
// inline assembly (the carry-out operand lands in a scalar register pair the
// result ignores).
template <uint32_t CLO, uint32_t CHI>
__device__ __forceinline__ uint64_t mul_const64(uint64_t z) {
    const uint32_t lo = (uint32_t)z;
    const uint32_t hi = (uint32_t)(z >> 32);
    const uint32_t t = lo * CHI;
    uint64_t cross, prod, carry0, carry1;
    asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(cross), "=s"(carry0) : "v"(hi), "s"(CLO), "v"((uint64_t)t));
    asm("v_mad_u64_u32 %0, %1, %2, %3, 0" : "=v"(prod), "=s"(carry1) : "v"(lo), "s"(CLO));
    uint32_t res_hi;
    asm("v_add_u32_e32 %0, %1, %2" : "=v"(res_hi) : "v"((uint32_t)(prod >> 32)), "v"((uint32_t)cross));
    return ((uint64_t)res_hi << 32) | (uint32_t)prod;
}

// The mixing function applied after the generator's first addition.
__device__ __forceinline__ uint64_t splitmix_mix(uint64_t z) {
    z = mul_const64<(uint32_t)kMul1, (uint32_t)(kMul1 >> 32)>(z ^ (z >> 30));
    z = mul_const64<(uint32_t)kMul2, (uint32_t)(kMul2 >> 32)>(z ^ (z >> 27));
    return z ^ (z >> 31);
}

// splitmix64 of  word ^ (index | Tag << 56)  for a word of array Tag at flat
// index `index`.  Indices stay below 2^56 (the host rejects larger ones) and
// a word has 32 bits, so the tag bits meet only zeros on both sides:
//   word ^ (index | Tag << 56) = (word ^ index) + (Tag << 56)
// and the tag folds into the constant the generator adds first,
//   z = (word ^ index) + (gamma + (Tag << 56))  mod 2^64.
template <uint32_t Tag>
__device__ __forceinline__ uint64_t hash_word(uint32_t word, uint64_t index) {
    static_assert(Tag < 4, "array tags 0..3");
    constexpr uint64_t kAdd = kGamma + ((uint64_t)Tag << 56);
    return splitmix_mix(((uint64_t)word ^ index) + kAdd);
}

// A wave-uniform value, in scalar registers.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint64_t uniform(uint64_t x) {
    return ((uint64_t)uniform((uint32_t)(x >> 32)) << 32) | uniform((uint32_t)x);
}

// The indices of the digest words of one vector tile, as seen by one lane:
// word `off` of the lane sits at flat index first + off.
//
// IndexAny: plain 64-bit indices, valid for every tile.
struct IndexAny {
    uint64_t first;  // index of the lane's first word
    __device__ __forceinline__ IndexAny(uint64_t tile_first, uint32_t lane_off) : first(tile_first + lane_off) {}
    template <uint32_t Tag>
    __device__ __forceinline__ uint64_t hash(uint32_t word, uint32_t off) const {
        return hash_word<Tag>(word, first + off);
    }
};

// The rest of the mix once the first round's product is known as
// prod + (cross << 32) (prod the full 64-bit product of the low halves with
// the first round's addend folded in, cross the low half of the cross
// term): the high half takes cross with one VOP2 add, then the second
// xor-shift and multiply and the final xor-shift.
__device__ __forceinline__ uint64_t mix_after_first_round(uint64_t prod, uint32_t cross) {
    uint32_t res_hi;
    asm("v_add_u32_e32 %0, %1, %2" : "=v"(res_hi) : "v"((uint32_t)(prod >> 32)), "v"(cross));
    uint64_t z = ((uint64_t)res_hi << 32) | (uint32_t)prod;
    z = z ^ (z >> 27);
    {
        constexpr uint32_t c2lo = (uint32_t)kMul2, c2hi = (uint32_t)(kMul2 >> 32);
        const uint32_t zl = (uint32_t)z, zh = (uint32_t)(z >> 32);
        const uint32_t t = zl * c2hi;
        uint64_t cr, pr, cy0, cy1;
        asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(cr), "=s"(cy0) : "v"(zh), "s"(c2lo), "v"(((uint64_t)zh << 32) | t));
        asm("v_mad_u64_u32 %0, %1, %2, %3, 0" : "=v"(pr), "=s"(cy1) : "v"(zl), "s"(c2lo));
        uint32_t rh;
        asm("v_add_u32_e32 %0, %1, %2" : "=v"(rh) : "v"((uint32_t)(pr >> 32)), "v"((uint32_t)cr));
        z = ((uint64_t)rh << 32) | (uint32_t)pr;
    }
    return z ^ (z >> 31);
}

// (h ^ (h >> 30)) * c mod 2^32 of wave-uniform h and c, on the scalar unit
// (left to itself the compiler forms such per-tile constants with VALU
// instructions, because their uses want VGPRs).
__device__ __forceinline__ uint32_t scalar_xorshift30_mul(uint32_t h, uint32_t c) {
    uint32_t r;
    asm("s_lshr_b32 %0, %1, 30\n\ts_xor_b32 %0, %0, %1\n\ts_mul_i32 %0, %0, %2" : "=&s"(r) : "s"(h), "s"(c) : "scc");
    return r;
}

// IndexHi32: for a tile whose indices all share their upper 32 bits `hi`
// (every tile but one that crosses a multiple of 2^32).  With index = hi:lo
// the word only meets the low half, so
//   z = (word ^ index) + gamma_k = zext(x) + G_k,   x = word ^ lo,
// where gamma_k = gamma + (k << 56) is the tagged constant above and
// G_k = (hi << 32) + gamma_k is one wave-uniform 64-bit value per tag.  Its
// low half is gamma's (the same for every tile and tag), so z's halves are
//   z_lo = x + G_lo (carry c),   z_hi = G_hi + c,
// and z_hi takes one of two values.  The first mixing round then reads the
// carry instead of a 64-bit value:
//   z ^ (z >> 30):  lo1 = z_lo ^ alignbit(z_hi, z_lo, 30),
//                   hi1 = z_hi ^ (z_hi >> 30), one of H_0, H_1 (c = 0, 1);
//   times C1 = CHI:CLO, low 64 bits: lo1 * CLO + ((lo1 * CHI + hi1 * CLO) << 32),
// and hi1 * CLO is one of K_0, K_1 = H_c * CLO mod 2^32.  So the product is
//   prod  = lo1 * CLO + (K_0 << 32)          v_mad_u64_u32, scalar addend
//   cross = lo1 * CHI + (c ? K_1 - K_0 : 0)  v_mad_u64_u32, low half used
//   z1    = prod + (cross << 32)             v_add_u32 on the high half
// with the carry, z_hi and the select taken by three VOP2 instructions that
// share the carry in VCC.  Against the plain round this trades a 64-bit
// shift, a multiply and the 64-bit index add (five VOP3 instructions) for
// three VOP3 and two more VOP2 ones; the later rounds are unchanged.
struct IndexHi32 {
    static constexpr uint32_t kGammaLo = (uint32_t)kGamma;
    uint32_t lo;        // low half of the lane's first index
    uint32_t ghi[4];    // G_hi per tag
    uint32_t kdiff[4];  // K_1 - K_0 per tag
    uint64_t k0hi[4];   // K_0 << 32 per tag
    __device__ __forceinline__ IndexHi32(uint64_t tile_first, uint32_t lane_off)
        : lo((uint32_t)tile_first + lane_off) {
        constexpr uint32_t clo = (uint32_t)kMul1;
        const uint64_t high = tile_first & 0xFFFFFFFF00000000ull;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t h = (uint32_t)((high + kGamma + ((uint64_t)k << 56)) >> 32);
            const uint32_t h1 = h + 1u;
            // wave-uniform per tile: scalar unit, then one copy into VGPRs
            const uint32_t k0 = scalar_xorshift30_mul(h, clo);
            const uint32_t k1 = scalar_xorshift30_mul(h1, clo);
            ghi[k] = h;
            kdiff[k] = k1 - k0;
            k0hi[k] = (uint64_t)k0 << 32;
        }
    }
    template <uint32_t Tag>
    __device__ __forceinline__ uint64_t hash(uint32_t word, uint32_t off) const {
        static_assert(Tag < 4, "array tags 0..3");
        constexpr uint32_t clo = (uint32_t)kMul1, chi = (uint32_t)(kMul1 >> 32);
        const uint32_t x = word ^ (lo + off);
        uint32_t zlo, zhi, ksel;
        // VCC carries c from the add to the select and to z_hi; a VALU write
        // of VCC needs two wait states before a VALU reads it as a lane mask.
        asm("v_add_co_u32_e32 %0, vcc, %3, %4\n\t"
            "s_nop 1\n\t"
            "v_cndmask_b32_e32 %1, 0, %5, vcc\n\t"
            "v_addc_co_u32_e32 %2, vcc, 0, %6, vcc"
            : "=&v"(zlo), "=&v"(ksel), "=v"(zhi)
            : "s"(kGammaLo), "v"(x), "v"(kdiff[Tag]), "v"(ghi[Tag])
            : "vcc");
        const uint32_t lo1 = zlo ^ __builtin_amdgcn_alignbit(zhi, zlo, 30);
        uint64_t prod, cross, carry0, carry1;
        asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(prod), "=s"(carry0) : "v"(lo1), "v"(clo), "s"(k0hi[Tag]));
        // Only cross's low half is used, so the addend's high half may hold
        // anything: z_hi, which sits beside the select in the register pair.
        asm("v_mad_u64_u32 %0, %1, %2, %3, %4"
            : "=v"(cross), "=s"(carry1)
            : "v"(lo1), "s"(chi), "v"(((uint64_t)zhi << 32) | ksel));
        return mix_after_first_round(prod, (uint32_t)cross);
    }
};

// IndexLo16: for a tile of 16-bit words (BF16 state, the bf16 working copy)
// whose indices all share bits 16..63.  There x = word ^ lo = A + v with
// A = lo & 0xFFFF0000 the same for the whole tile and v < 2^16, so with
// B = A + G_lo = c0 * 2^32 + B_lo (wave-uniform):
//   z_lo = x + G_lo = B_lo + v,   z_hi = G_hi + c0,
// provided B_lo + v never carries out of 32 bits (B_lo <= 0xFFFF0000).  If
// moreover no carry reaches bit 30 ((B_lo mod 2^30) <= 0x3FFF0000), the top
// two bits of z_lo are those of B_lo, T = B_lo >> 30, so the first mixing
// round is
//   lo1 = z_lo ^ (T | z_hi << 2) = (x + G_lo) ^ U_k,   hi1 = H_k,
//   z1  = lo1 * CLO + ((lo1 * CHI + H_k * CLO) << 32),
// with U_k, H_k and K_k = H_k * CLO wave-uniform per tag: an add, an xor, a
// multiply-add with the scalar addend K_k << 32, a multiply and an add, two
// VOP3 instructions against three (and three fewer VALU instructions) in
// IndexHi32, and no carry to pass.  The two checks fail only for A in
// {0x00B50000, 0x40B50000, 0x80B50000, 0xC0B50000}; such a tile, and one that
// crosses a multiple of 2^16, takes IndexHi32 or IndexAny.
struct IndexLo16 {
    static constexpr uint32_t kGammaLo = (uint32_t)kGamma;
    uint32_t lo;       // low half of the lane's first index
    uint32_t u[4];     // U_k per tag
    uint64_t khi[4];   // K_k << 32 per tag
    // Whether the tile of n indices from `first` on may take this form
    // (wave-uniform).
    static __device__ __forceinline__ bool applies(uint64_t first, uint32_t n) {
        if ((first >> 16) != ((first + n - 1) >> 16)) {
            return false;
        }
        const uint32_t b_lo = ((uint32_t)first & 0xFFFF0000u) + kGammaLo;
        return b_lo <= 0xFFFF0000u && (b_lo & 0x3FFFFFFFu) <= 0x3FFF0000u;
    }
    __device__ __forceinline__ IndexLo16(uint64_t tile_first, uint32_t lane_off)
        : lo((uint32_t)tile_first + lane_off) {
        constexpr uint32_t clo = (uint32_t)kMul1;
        const uint64_t b = (uint64_t)((uint32_t)tile_first & 0xFFFF0000u) + kGammaLo;
        const uint32_t c0 = (uint32_t)(b >> 32);
        const uint32_t t = (uint32_t)b >> 30;
        const uint32_t hi = (uint32_t)(tile_first >> 32);
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t zhi = hi + (uint32_t)(kGamma >> 32) + (k << 24) + c0;
            u[k] = (zhi << 2) | t;
            khi[k] = (uint64_t)scalar_xorshift30_mul(zhi, clo) << 32;
        }
    }
    template <uint32_t Tag>
    __device__ __forceinline__ uint64_t hash(uint32_t word, uint32_t off) const {
        static_assert(Tag < 4, "array tags 0..3");
        constexpr uint32_t clo = (uint32_t)kMul1, chi = (uint32_t)(kMul1 >> 32);
        const uint32_t x = word ^ (lo + off);
        uint32_t zlo;
        asm("v_add_u32_e32 %0, %1, %2" : "=v"(zlo) : "s"(kGammaLo), "v"(x));
        const uint32_t lo1 = zlo ^ u[Tag];
        uint64_t prod, carry0;
        asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(prod), "=s"(carry0) : "v"(lo1), "v"(clo), "s"(khi[Tag]));
        return mix_after_first_round(prod, lo1 * chi);
    }
};

// Whether the `count` indices from `first` on share their upper 32 bits.
__device__ __forceinline__ bool same_high_half(uint64_t first, uint64_t count) {
    return (first >> 32) == ((first + count - 1) >> 32);
}

// ---------------------------------------------------------------------------
// AdamW on one element, in the contract's order.  With -ffp-contract=off and
// no fast-math flags every +, -, * below is one IEEE binary32 operation
// rounded to nearest even, '/' is the correctly rounded division, and
// __builtin_sqrtf is lowered to the correctly rounded square root (the
// -fhip-fp32-correctly-rounded-divide-sqrt default).  HIP's __fsqrt_rn is
// NOT used: unless OCML_BASIC_ROUNDED_OPERATIONS is defined it maps to the
// hardware's approximate v_sqrt_f32.  The update is split in two: the
// moments, then the bias-corrected step, so that a tile can pick the form of
// the square root once for all its elements (see sqrt_rn_in_range).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void adamw_moments(float& p, float g, float& m, float& v, const StepScalars& s) {
    const float p_dec = p * s.decay;
    const float m_keep = s.beta1 * m;
    const float m_push = s.omb1 * g;
    const float m_new = m_keep + m_push;
    const float g_sq = g * g;
    const float v_keep = s.beta2 * v;
    const float v_push = s.omb2 * g_sq;
    const float v_new = v_keep + v_push;
    p = p_dec;
    m = m_new;
    v = v_new;
}

// Correctly rounded square root of x in [2^-96, +inf).  The hardware root
// s = v_sqrt_f32(x) is within one ulp of sqrt(x) there (so is the compiler's
// full sequence built on it), so the correctly rounded root is s or one of
// its neighbours s_dn, s_up (bit patterns minus and plus one), and two exact
// residuals decide which (the rounding test for square roots by fused
// multiply-add, as in Markstein's and Goldschmidt-style refinements):
//   x <= s_dn * s  => sqrt(x) lies below the midpoint of s_dn and s
//                     (the geometric mean is below the arithmetic one);
//   x >  s * s_up  => sqrt(x) lies above the midpoint of s and s_up: the
//                     squared midpoint exceeds s * s_up by ulp^2 / 4, and
//                     no binary32 x falls in that gap (x's grid near s^2 is
//                     at least 2^22 of those units);
//   otherwise s.
// The residuals x - s_dn*s and x - s_up*s are computed by one FMA each; for
// x >= 2^-96 they are multiples of 2^-142, so their signs come out exact
// (denormals are kept).  The compiler's full sequence adds a rescaling of
// inputs below 2^-96 and a class test for 0 and infinity; a tile whose
// inputs all lie in [2^-96, +inf) takes this form (a wave-uniform branch),
// any other tile the full one, with the same bits.
__device__ __forceinline__ bool sqrt_rn_in_range(float x) {
    return (__float_as_uint(x) - 0x0F800000u) < (0x7F800000u - 0x0F800000u);
}

__device__ __forceinline__ float sqrt_rn_in_range_root(float x) {
    const float s = __builtin_amdgcn_sqrtf(x);
    const float s_dn = __uint_as_float(__float_as_uint(s) - 1u);
    const float s_up = __uint_as_float(__float_as_uint(s) + 1u);
    const float r_dn = __builtin_fmaf(-s_dn, s, x);
    const float r_up = __builtin_fmaf(-s_up, s, x);
    const float t = r_dn <= 0.0f ? s_dn : s;
    return r_up > 0.0f ? s_up : t;
}

template <bool InRange>
__device__ __forceinline__ float adamw_step(float p_dec, float m_new, float v_new, const StepScalars& s) {
    const float root = InRange ? sqrt_rn_in_range_root(v_new) : __builtin_sqrtf(v_new);
    const float den = root * s.rs_bc2 + s.eps;
    const float ratio = m_new / den;
    const float step = s.step_size * ratio;
    return p_dec - step;
}

__device__ __forceinline__ void adamw(float& p, float g, float& m, float& v, const StepScalars& s) {
    adamw_moments(p, g, m, v, s);
    p = adamw_step<false>(p, m, v, s);
}

// The bias-corrected steps of all n elements of a lane's share of a tile
// (p holds p*decay, m and v the new moments), with the short square root
// when every v of the wave is in its range.
template <int N>
__device__ __forceinline__ void adamw_steps(float (&p)[N], const float (&m)[N], const float (&v)[N],
                                            const StepScalars& s) {
    bool in_range = true;
#pragma unroll
    for (int i = 0; i < N; ++i) in_range = in_range && sqrt_rn_in_range(v[i]);
    if (__builtin_amdgcn_ballot_w64(!in_range) == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            p[i] = adamw_step<true>(p[i], m[i], v[i], s);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            p[i] = adamw_step<false>(p[i], m[i], v[i], s);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// binary32 -> bfloat16, round to nearest even; NaN stays a quiet NaN with
// its sign and top payload bits.  The rule, on the bits u of x:
//   NaN:       (u >> 16) | 0x0040
//   otherwise: (u + 0x7FFF + ((u >> 16) & 1)) >> 16
// gfx950's v_cvt_pk_bf16_f32 computes exactly this, two values per
// instruction, so the kernels use it: a GPU test sends all 2^32 patterns
// through the commit as weights (p' = p * 1 - 0) and compares the bf16 copy
// with this rule applied to the GPU's own p', NaNs included.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t to_bf16x2(float lo, float hi) {
    const f32x2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

__device__ __forceinline__ uint32_t to_bf16(float x) { return to_bf16x2(x, 0.0f) & 0xFFFFu; }
__device__ __forceinline__ float widen_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float widen_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// The larger, per half, of `most` and words * scale - from.
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2_t max_offset(u16x2_t most, uint32_t words, uint16_t scale, uint16_t from) {
    const u16x2_t w = __builtin_bit_cast(u16x2_t, words);
    return __builtin_elementwise_max(most, (u16x2_t)(w * scale - from));
}
__device__ __forceinline__ bool below(u16x2_t x, uint16_t limit) { return std::max(x.x, x.y) < limit; }

// AdamW on a lane's 2 * N elements of one row of BF16 state, pairs of bf16 words.
//
// The exact step spends 19 of its instructions per element on a correctly rounded
// square root and division, of which the rounding to bf16 keeps hardly anything.
// So the step s = RN(step_size * RN(m / den)) is bracketed first: with the hardware's
// root and reciprocal (each within one bit pattern of the correctly rounded one)
//   s' = step_size * RN(m * rcp(RN(root' * rs_bc2 + eps))),
// and unless something under- or overflows, s' and s differ by at most
// 5 * 2^-24 (the roundings in s) + 8 * 2^-24 (two of 3 * 2^-24 and two of 2^-24 in s').
// With 2^-24 for the rounding of step_size * (1 -+ 2^-20) that is less than 2^-20.
// Rounding is monotone, to binary32 and on to bf16, so RN(p - s) lies between the two
// fused p - RN(m * ..) * RN(step_size * (1 -+ 2^-20)), and where these round to the same
// bf16 word that is the result.  Nothing under- or overflows to any effect if
//   2^-40 <= step_size <= 2^40 and eps <= 2^100  (wave-uniform),
//   2^-95 <= v < inf: den and its reciprocal are normal numbers;
//   2^-50 <= |p'| < 2^20: as both ends round to one word, |s'| < 2^60, so that m / den
//     does not overflow; what underflow adds to s is below 2^-108, no more than 2^-25
//     of s' where |s'| >= 2^-83, and where |s'| is less both ends and RN(p - s) are p.
// A NaN or an infinity anywhere leaves p' or v outside these ranges.  A row of a wave
// with an element that fails takes the exact form.
//
// Bound by VALU issue and the clock it leaves: 79.9 instructions per element (counted)
// against 94.8 with the exact step.  453M elements 1187 -> 1120 us (5.7 TB/s), 76M 202 ->
// 186, 6M 20.8 -> 19.0; fewer tiles in flight, 4 KB tiles and longer runs per XCD, which
// the HBM-bound commits want, made no difference.
template <int N>
__device__ __forceinline__ void adamw_row_bf16(uint32_t (&P)[N], uint32_t (&G)[N], uint32_t (&M)[N],
                                               uint32_t (&V)[N], const StepScalars& s) {
    if (s.step_size >= 0x1p-40f && s.step_size <= 0x1p40f && s.eps <= 0x1p100f) {
        constexpr uint16_t kVFrom = 0x1000, kVLimit = 0x7F80 - kVFrom;  // 2^-95 up to infinity
        constexpr uint16_t kPFrom = 0x2680, kPLimit = 0x4980 - kPFrom;  // 2^-50 up to 2^20, signs shifted out
        const float size_lo = s.step_size * (1.0f - 0x1p-20f), size_hi = s.step_size * (1.0f + 0x1p-20f);
        u16x2_t v_most = {0, 0}, p_most = {0, 0};
        uint32_t differ = 0;
        uint32_t p_new[N], m_new[N], v_new[N];
        auto ends = [&](float p, float g, float& m, float& v, float& near, float& far) {
            adamw_moments(p, g, m, v, s);
            const float den = __builtin_fmaf(__builtin_amdgcn_sqrtf(v), s.rs_bc2, s.eps);
            const float ratio = m * __builtin_amdgcn_rcpf(den);
            near = __builtin_fmaf(ratio, -size_lo, p);
            far = __builtin_fmaf(ratio, -size_hi, p);
        };
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float near[2], far[2], m[2] = {widen_lo(M[i]), widen_hi(M[i])}, v[2] = {widen_lo(V[i]), widen_hi(V[i])};
            ends(widen_lo(P[i]), widen_lo(G[i]), m[0], v[0], near[0], far[0]);
            ends(widen_hi(P[i]), widen_hi(G[i]), m[1], v[1], near[1], far[1]);
            p_new[i] = to_bf16x2(near[0], near[1]);
            m_new[i] = to_bf16x2(m[0], m[1]);
            v_new[i] = to_bf16x2(v[0], v[1]);
            differ |= p_new[i] ^ to_bf16x2(far[0], far[1]);
            p_most = max_offset(p_most, p_new[i], 2, 2 * kPFrom);
            v_most = max_offset(v_most, v_new[i], 1, kVFrom);
            __builtin_amdgcn_sched_barrier(0);
        }
        const uint32_t fails = differ | (below(p_most, 2 * kPLimit) ? 0u : 1u) | (below(v_most, kVLimit) ? 0u : 1u);
        if (__builtin_amdgcn_ballot_w64(fails != 0) == 0) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                P[i] = p_new[i];
                M[i] = m_new[i];
                V[i] = v_new[i];
            }
            return;
        }
    }
    float p[2 * N], m[2 * N], v[2 * N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        // (opaque, or the moments from above are kept instead of formed again)
        asm volatile("" : "+v"(P[i]), "+v"(G[i]), "+v"(M[i]), "+v"(V[i]));
        p[2 * i] = widen_lo(P[i]);
        p[2 * i + 1] = widen_hi(P[i]);
        m[2 * i] = widen_lo(M[i]);
        m[2 * i + 1] = widen_hi(M[i]);
        v[2 * i] = widen_lo(V[i]);
        v[2 * i + 1] = widen_hi(V[i]);
        adamw_moments(p[2 * i], widen_lo(G[i]), m[2 * i], v[2 * i], s);
        adamw_moments(p[2 * i + 1], widen_hi(G[i]), m[2 * i + 1], v[2 * i + 1], s);
    }
    adamw_steps<2 * N>(p, m, v, s);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        P[i] = to_bf16x2(p[2 * i], p[2 * i + 1]);
        M[i] = to_bf16x2(m[2 * i], m[2 * i + 1]);
        V[i] = to_bf16x2(v[2 * i], v[2 * i + 1]);
    }
}

// ---------------------------------------------------------------------------
// workgroup sum of a 64-bit value; result valid in thread 0
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t block_sum(uint64_t x, uint64_t* lds) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        x += __shfl_xor(x, off, 64);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        lds[wave] = x;
    }
    __syncthreads();
    uint64_t r = 0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
            r += lds[w];
        }
    }
    return r;
}

// ---------------------------------------------------------------------------
// result slots: handing in the workgroups' shares
//
// A node is two workspace words that gather n shares x < 2^64:
//   word 0  count in bits 44..63, sum of the shares' low 24 bits below it;
//   word 1  sum of the high 40 bits in bits 24..63, count below it.
// Each share is added with one relaxed atomic per word.  A word carries its
// own count, so the arrival that finds n - 1 others there holds the word's
// complete sum: it needs no ordering between different words, hence no fence
// (at agent scope a release or acquire writes back or invalidates the XCD's
// L2).  n <= 2^20 fits: 2^20 sums of 24 bits stay below 2^44, the high sum is
// needed mod 2^40 only and drops off the top, and so may the low word's count
// on its last arrival.  The last arrival at word 0 passes the carry out of 24
// bits on to word 1, which therefore waits for n + 1 arrivals; the last
// arrival at each word sets it back to zero and writes its bytes of the result
// (3 and 5 of them: no thread ever holds all 64 bits beside a count).
//
// A result slot has one node its tiles arrive at when they are few, else
// kLanes of them (256 bytes apart, so that neighbouring workgroups do not queue
// on one address) whose last arrivals go on to the slot's own node; there the
// count of word 0 sits in bits 56..63, since a lane's sum has up to 44 bits.
// With per-segment results the tiles also arrive at the nodes of the total,
// in the same instructions.
//
// There are two sets of nodes.  A call uses one and clears the other one
// (which is clear already unless the caller broke its word about the
// workspace), so that a caller who alternates them has right digests again one
// call after a wrong one.
//
// Against a launch that sums the lanes behind the tiles, the last workgroup's
// two or three dependent atomics take about 0.6 us each where that launch took
// 2-3 us of the GPU and 2.5 us of the host.
// ---------------------------------------------------------------------------
constexpr uint32_t kLowBits = 24;
constexpr uint64_t kLowMask = (1ull << kLowBits) - 1;
constexpr int kCountAtTiles = 44;  // where word 0's count begins in a node fed by tiles
constexpr int kCountAtLanes = 56;  // and in one fed by lanes

// Tiles of a result from which on its shares are spread over kLanes nodes: one
// address takes about 11 ns per atomic, the further level 0.6 us once.
constexpr uint32_t kSpreadTiles = 64;

__device__ __forceinline__ uint64_t node_add(uint64_t* word, uint64_t x) {
    return __hip_atomic_fetch_add(word, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void node_clear(uint64_t* word) {
    __hip_atomic_store(word, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One tile hands in its share s to the result at dst, as number `index` of the
// result's n tiles: lanes 0 and 1 of one wave, for word 0 and word 1, in the same
// instructions (everything but s and the words themselves is wave-uniform: the
// 60 VALU instructions that this took at first were 1% of a state digest).
// Lane l's node is at lanes + l * kLaneStride.  (A wait for an atomic's result
// waits for the stores before it too, so every store is issued behind the next
// atomic.)
__device__ __forceinline__ void hand_in(uint64_t* lanes, uint64_t* own, uint64_t* dst, uint32_t n, uint32_t index,
                                        uint64_t s) {
    const uint32_t word = threadIdx.x & 1;
    const bool low = word == 0;
    const bool spread = n > kSpreadTiles;
    const uint32_t l = index & (kLanes - 1);
    uint64_t* const first = spread ? lanes + l * kLaneStride : own;
    const uint32_t in_first = spread ? (n - l + kLanes - 1) / kLanes : n;  // the tiles that arrive there
    const uint32_t in_own = spread ? (uint32_t)kLanes : n;
    // this word's part of a sum, and one arrival
    auto part_of = [&](uint64_t x, int count_at) {
        const uint64_t low_part = x & ((1ull << count_at) - 1), high_part = x & ~kLowMask;
        return low ? low_part : high_part;
    };
    auto arrivals = [&](uint64_t x, int count_at) {
        const uint32_t at_low = (uint32_t)(x >> count_at), at_high = (uint32_t)x & (uint32_t)kLowMask;
        return low ? at_low : at_high;
    };
    uint64_t part = part_of(s, kLowBits);
    uint64_t old = node_add(first + word, part + (low ? 1ull << kCountAtTiles : 1ull));
    // (word 1 of the own node gets word 0's carry besides)
    if (arrivals(old, kCountAtTiles) != (low || spread ? in_first - 1 : in_first)) return;
    part += part_of(old, kCountAtTiles);
    if (spread) {
        old = node_add(own + word, part + (low ? 1ull << kCountAtLanes : 1ull));
        node_clear(first + word);
        if (arrivals(old, kCountAtLanes) != (low ? in_own - 1 : in_own)) return;
        part += part_of(old, kCountAtLanes);
    }
    uint8_t* const b = reinterpret_cast<uint8_t*>(dst);
    if (low) {
        const uint64_t carry = part & ~kLowMask;
        old = node_add(own + 1, carry + 1u);
        node_clear(own);
        *reinterpret_cast<uint16_t*>(b) = (uint16_t)part;
        b[2] = (uint8_t)(part >> 16);
        if ((uint32_t)(old & kLowMask) != in_own) return;
        part = (old & ~kLowMask) + carry;
    }
    node_clear(own + 1);
    b[3] = (uint8_t)(part >> kLowBits);
    *reinterpret_cast<uint32_t*>(b + 4) = (uint32_t)(part >> 32);
}

// The nodes of a slot (of the total too, with slot 0) in the set that this
// call does not use.
__device__ __forceinline__ void clear_other_set(const Results& r, uint32_t slot) {
    constexpr uint32_t kNodes = kNodesPerLane / 2;
    if (threadIdx.x < kLanes * kNodes) {
        uint64_t* node = r.words + ((uint64_t)slot * kLanes + threadIdx.x / kNodes) * kLaneStride +
                         threadIdx.x % kNodes * 4 + (r.set ^ 1u) * 2;
        node_clear(node);
        node_clear(node + 1);
    }
}

// ---------------------------------------------------------------------------
// HBM access: raw buffer instructions on a per-tile resource (base address in
// scalar registers, 32-bit byte offset per lane), with the non-temporal cache
// policy on loads and stores -- every byte is touched exactly once.
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kRsrcWord3 = 0x00020000;  // raw, untyped buffer (gfx9 family)
constexpr int kNonTemporal = 2;         // cache-policy 'nt' bit

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, kRsrcWord3);
}

// The whole byte offset travels in the per-lane VGPR offset and the scalar
// offset field stays the literal 0.  That matters for stores wider than 8
// bytes: their data VGPRs must not be overwritten by the very next VALU
// instruction (one wait state), and the compiler only guards that hazard
// when the scalar offset is not a register.  With a register scalar offset a
// following VALU write was seen to corrupt the first dword of the stored
// vector.
__device__ __forceinline__ u32x4 load16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kNonTemporal);
}
__device__ __forceinline__ void store16(u32x4 x, __amdgpu_buffer_rsrc_t r, uint32_t off) {
    __builtin_amdgcn_raw_buffer_store_b128(x, r, (int)off, 0, kNonTemporal);
}
__device__ __forceinline__ u32x2 load8(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, kNonTemporal);
}
__device__ __forceinline__ void store8(u32x2 x, __amdgpu_buffer_rsrc_t r, uint32_t off) {
    __builtin_amdgcn_raw_buffer_store_b64(x, r, (int)off, 0, kNonTemporal);
}

// A vector of eight or four 16-bit words.
template <int Vec>
struct Words16;
template <>
struct Words16<8> {
    typedef u32x4 type;
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, uint32_t off) { return load16(r, off); }
    static __device__ __forceinline__ void store(type x, __amdgpu_buffer_rsrc_t r, uint32_t off) { store16(x, r, off); }
};
template <>
struct Words16<4> {
    typedef u32x2 type;
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, uint32_t off) { return load8(r, off); }
    static __device__ __forceinline__ void store(type x, __amdgpu_buffer_rsrc_t r, uint32_t off) { store8(x, r, off); }
};

// ---------------------------------------------------------------------------
// one element, element-wise path (ragged tails, misaligned segments)
// ---------------------------------------------------------------------------
template <Mode M>
constexpr bool kCommits = binary32_commit(M);

// Kernels whose tiles may have several passes.  (The state digest's usual kernel
// without the loop: with it, one pass a tile, 76M elements took 156 us against 146.)
template <Mode M, Form F>
constexpr bool kManyPasses = M == Mode::StateDigest ? F == Form::Long
                                                    : F == Form::Usual && (M == Mode::Bf16Digest || M == Mode::DigestBf16State);

// Kernels whose whole tiles branch around everything that only a tile with ragged ends
// needs, which the others form in every tile.  us per state digest without / with it (and
// of the form in which no tile had such ends): 76M elements 154.4 / 153.6 (154.2), 220M
// 440.7 / 438.4 (437.7), 400M 801.3 / 797.1 (794.8).  Every other kernel is slower with it:
// BF16 commit of 9.3M 26.7 -> 28.4 (25 scalar registers spilled instead of 10), guard,
// digests and boundaries of a hundred and more short segments up to 8%.
template <Mode M, Form F>
constexpr bool kWholeApart = M == Mode::StateDigest && F != Form::Small;

// Modes whose digest words have 16 bits (the short IndexLo16 form applies).
template <Mode M>
constexpr bool kWords16 = (M == Mode::Bf16Digest || M == Mode::CommitBf16State || M == Mode::DigestBf16State);

template <Mode M>
__device__ __forceinline__ uint64_t do_scalar(const Arrays& a, uint64_t e, const StepScalars& sc) {
    const uint64_t idx = a.goff + e;
    if constexpr (M == Mode::Bf16Digest) {
        return hash_word<kTagB>(a.b[e], idx);
    } else if constexpr (M == Mode::GradGuard) {
        return __float_as_uint(a.g[e]) != 0u ? 1u : 0u;
    } else {
        float p = a.p[e];
        float m = a.m[e];
        float v = a.v[e];
        if constexpr (kCommits<M>) {
            adamw(p, a.g[e], m, v, sc);
            a.p[e] = p;
            a.m[e] = m;
            a.v[e] = v;
            a.b[e] = (uint16_t)to_bf16(p);
            if constexpr (M == Mode::CommitZeroGrad) {
                a.g_zero[e] = 0.0f;
            }
        }
        return hash_word<kTagP>(__float_as_uint(p), idx) + hash_word<kTagM>(__float_as_uint(m), idx) +
               hash_word<kTagV>(__float_as_uint(v), idx);
    }
}

// ---------------------------------------------------------------------------
// one pass of a tile, whose start is 16-byte aligned in every fp32 array (8-byte in the
// bf16 array): Rows rows of kBlock vectors per array.  Row u, lane t holds
// elements e0 + (u*kBlock + t)*Vec .. + Vec - 1 (Vec is 4 in the modes that read
// fp32 arrays, 16-byte vectors).  Masked: one row of which only the
// first nvec vectors exist; the buffer range check drops the others' loads and
// stores (whole vectors, since the range ends with one), and their hashes are
// not counted (and go one element after another: it is not to cost the full
// tiles registers).
// ---------------------------------------------------------------------------
template <Mode M, typename Ix, int Vec, int Rows, bool Masked>
__device__ __forceinline__ uint64_t do_tile_vec(const Arrays& a, uint64_t e0, uint32_t nvec, const StepScalars& sc) {
    static_assert(Vec == 4 || M == Mode::Bf16Digest, "16-byte vectors of fp32");
    constexpr uint32_t kRow32 = kBlock * Vec * 4;  // bytes of one fp32 row
    constexpr uint32_t kRow16 = kBlock * Vec * 2;  // bytes of one bf16 row
    static_assert(!Masked || Rows == 1, "a masked tile is one row");
    const uint32_t bytes32 = Masked ? nvec * Vec * 4 : Rows * kRow32;
    const uint32_t bytes16 = Masked ? nvec * Vec * 2 : Rows * kRow16;
    const uint32_t lane32 = threadIdx.x * Vec * 4;
    const uint32_t lane16 = threadIdx.x * Vec * 2;
    const Ix ix(a.goff + e0, threadIdx.x * Vec);  // word k of this lane: index + k
    uint64_t acc = 0;
    if constexpr (M == Mode::GradGuard) {
        const auto rg = tile_rsrc(a.g + e0, bytes32);
        u32x4 G[Rows];
#pragma unroll
        for (int u = 0; u < Rows; ++u) {
            G[u] = load16(rg, lane32 + u * kRow32);
        }
#pragma unroll
        for (int u = 0; u < Rows; ++u) {
#pragma unroll
            for (int j = 0; j < Vec; ++j) {
                acc += G[u][j] != 0u ? 1u : 0u;  // a dropped load reads zero
            }
        }
        return acc;
    } else if constexpr (M == Mode::Bf16Digest) {
        const auto rb = tile_rsrc(a.b + e0, bytes16);
        typename Words16<Vec>::type W[Rows];
#pragma unroll
        for (int u = 0; u < Rows; ++u) {
            W[u] = Words16<Vec>::load(rb, lane16 + u * kRow16);
        }
#pragma unroll
        for (int u = 0; u < Rows; ++u) {
#pragma unroll
            for (int j = 0; j < Vec / 2; ++j) {
                const uint32_t o = u * kBlock * Vec + 2 * j;
                acc += ix.template hash<kTagB>(W[u][j] & 0xFFFFu, o) + ix.template hash<kTagB>(W[u][j] >> 16, o + 1);
                if constexpr (Masked) __builtin_amdgcn_sched_barrier(0);
            }
        }
        return Masked && threadIdx.x >= nvec ? 0 : acc;
    } else {
        const auto rp = tile_rsrc(a.p + e0, bytes32);
        const auto rm = tile_rsrc(a.m + e0, bytes32);
        const auto rv = tile_rsrc(a.v + e0, bytes32);
        u32x4 P[Rows], G[Rows], Mo[Rows], V[Rows];
#pragma unroll
        for (int u = 0; u < Rows; ++u) {
            P[u] = load16(rp, lane32 + u * kRow32);
            Mo[u] = load16(rm, lane32 + u * kRow32);
            V[u] = load16(rv, lane32 + u * kRow32);
        }
        if constexpr (kCommits<M>) {
            const auto rg = tile_rsrc(a.g + e0, bytes32);
#pragma unroll
            for (int u = 0; u < Rows; ++u) {
                G[u] = load16(rg, lane32 + u * kRow32);
            }
            if constexpr (M == Mode::CommitZeroGrad) {
                const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int u = 0; u < Rows; ++u) {
                    store16(zero, rg, lane32 + u * kRow32);
                }
            }
            const auto rb = tile_rsrc(a.b + e0, bytes16);
            // Bound by HBM: each row is updated and stored as soon as it is
            // ready, with the full square root (the short in-range form of the
            // BF16-state commit measured no faster here).
#pragma unroll
            for (int u = 0; u < Rows; ++u) {
                    float p[4], m[4], v[4];
#pragma unroll
                for (int j = 0; j < Vec; ++j) {
                    p[j] = __uint_as_float(P[u][j]);
                    m[j] = __uint_as_float(Mo[u][j]);
                    v[j] = __uint_as_float(V[u][j]);
                    adamw(p[j], __uint_as_float(G[u][j]), m[j], v[j], sc);
                    P[u][j] = __float_as_uint(p[j]);
                    Mo[u][j] = __float_as_uint(m[j]);
                    V[u][j] = __float_as_uint(v[j]);
                }
                store16(P[u], rp, lane32 + u * kRow32);
                store16(Mo[u], rm, lane32 + u * kRow32);
                store16(V[u], rv, lane32 + u * kRow32);
                u32x2 h;
                h.x = to_bf16x2(p[0], p[1]);
                h.y = to_bf16x2(p[2], p[3]);
                store8(h, rb, lane16 + u * kRow16);
            }
        }
#pragma unroll
        for (int u = 0; u < Rows; ++u) {
#pragma unroll
            for (int j = 0; j < Vec; ++j) {
                const uint32_t o = u * kBlock * Vec + j;
                acc += ix.template hash<kTagP>(P[u][j], o) + ix.template hash<kTagM>(Mo[u][j], o) +
                       ix.template hash<kTagV>(V[u][j], o);
                if constexpr (Masked) __builtin_amdgcn_sched_barrier(0);
            }
        }
        return Masked && threadIdx.x >= nvec ? 0 : acc;
    }
}

// ---------------------------------------------------------------------------
// BF16 state: vectors of Vec (eight or four) bf16 words per array; element 2j
// of a vector is the low half of its word j.
// ---------------------------------------------------------------------------
template <Mode M>
__device__ __forceinline__ uint64_t do_scalar(const ArraysBf16& a, uint64_t e, const StepScalars& sc) {
    const uint64_t idx = a.goff + e;
    uint32_t p = a.p[e];
    uint32_t m = a.m[e];
    uint32_t v = a.v[e];
    if constexpr (M == Mode::CommitBf16State) {
        float pf = widen_lo(p), mf = widen_lo(m), vf = widen_lo(v);
        adamw(pf, widen_lo(a.g[e]), mf, vf, sc);
        p = to_bf16(pf);
        m = to_bf16(mf);
        v = to_bf16(vf);
        a.p[e] = (uint16_t)p;
        a.m[e] = (uint16_t)m;
        a.v[e] = (uint16_t)v;
    }
    return hash_word<kTagP>(p, idx) + hash_word<kTagM>(m, idx) + hash_word<kTagV>(v, idx);
}

template <Mode M, int Vec, int Rows, bool Masked>
__device__ __forceinline__ uint64_t do_pass_bf16(const ArraysBf16& a, uint64_t e0, uint32_t nvec,
                                                 const StepScalars& sc) {
    static_assert(!Masked || Rows == 1, "a masked pass is one row");
    using W = Words16<Vec>;
    constexpr int kN = Vec / 2;  // words of a vector
    constexpr uint32_t kRowBytes = kBlock * Vec * 2;
    const uint32_t lane = threadIdx.x * Vec * 2;
    const uint32_t bytes = Masked ? nvec * Vec * 2 : Rows * kRowBytes;
    const auto rp = tile_rsrc(a.p + e0, bytes);
    const auto rm = tile_rsrc(a.m + e0, bytes);
    const auto rv = tile_rsrc(a.v + e0, bytes);
    uint32_t P[Rows][kN], G[Rows][kN], Mo[Rows][kN], V[Rows][kN];
    auto load = [&](uint32_t (&x)[kN], __amdgpu_buffer_rsrc_t rsrc, int r) {
        const auto w = W::load(rsrc, lane + r * kRowBytes);
#pragma unroll
        for (int j = 0; j < kN; ++j) x[j] = w[j];
    };
    auto store = [&](const uint32_t (&x)[kN], __amdgpu_buffer_rsrc_t rsrc, int r) {
        typename W::type w;
#pragma unroll
        for (int j = 0; j < kN; ++j) w[j] = x[j];
        W::store(w, rsrc, lane + r * kRowBytes);
    };
#pragma unroll
    for (int r = 0; r < Rows; ++r) {
        load(P[r], rp, r);
        load(Mo[r], rm, r);
        load(V[r], rv, r);
    }
    if constexpr (M == Mode::CommitBf16State) {
        const auto rg = tile_rsrc(a.g + e0, bytes);
#pragma unroll
        for (int r = 0; r < Rows; ++r) load(G[r], rg, r);
#pragma unroll
        for (int r = 0; r < Rows; ++r) {
            adamw_row_bf16<kN>(P[r], G[r], Mo[r], V[r], sc);
            store(P[r], rp, r);
            store(Mo[r], rm, r);
            store(V[r], rv, r);
        }
    }
    const uint64_t first = a.goff + e0;
    auto digest = [&](const auto& ix) {  // word k of this lane: index + k
        uint64_t acc = 0;
#pragma unroll
        for (int r = 0; r < Rows; ++r) {
#pragma unroll
            for (int j = 0; j < kN; ++j) {
                const uint32_t o = r * kBlock * Vec + 2 * j;
                // (opaque, or the halves of all words are taken apart, and kept, before
                // the branch on the index form)
                uint32_t p = P[r][j], m = Mo[r][j], v = V[r][j];
                asm volatile("" : "+v"(p), "+v"(m), "+v"(v));
                acc += ix.template hash<kTagP>(p & 0xFFFFu, o) + ix.template hash<kTagP>(p >> 16, o + 1) +
                       ix.template hash<kTagM>(m & 0xFFFFu, o) + ix.template hash<kTagM>(m >> 16, o + 1) +
                       ix.template hash<kTagV>(v & 0xFFFFu, o) + ix.template hash<kTagV>(v >> 16, o + 1);
                if constexpr (Masked) __builtin_amdgcn_sched_barrier(0);
            }
        }
        return acc;
    };
    if constexpr (Masked) {
        const uint64_t acc = digest(IndexAny(first, threadIdx.x * Vec));
        return threadIdx.x >= nvec ? 0 : acc;
    } else {
        constexpr uint32_t kPass = kBlock * Vec * Rows;
        if (IndexLo16::applies(first, kPass)) return digest(IndexLo16(first, threadIdx.x * Vec));
        if (same_high_half(first, kPass)) return digest(IndexHi32(first, threadIdx.x * Vec));
        return digest(IndexAny(first, threadIdx.x * Vec));
    }
}

// The whole pass, whatever index form it takes, and one row of whole vectors.
template <Mode M, int Vec, int Rows>
__device__ __forceinline__ uint64_t do_pass(const ArraysBf16& a, uint64_t e0, const StepScalars& sc) {
    return do_pass_bf16<M, Vec, Rows, false>(a, e0, 0, sc);
}
template <Mode M, int Vec>
__device__ __forceinline__ uint64_t do_row(const ArraysBf16& a, uint64_t e0, uint32_t nvec, const StepScalars& sc) {
    return do_pass_bf16<M, Vec, 1, true>(a, e0, nvec, sc);
}
template <Mode M, int Vec, int Rows>
__device__ __forceinline__ uint64_t do_pass(const Arrays& a, uint64_t e0, const StepScalars& sc) {
    constexpr uint32_t kPass = kBlock * Vec * Rows;
    // The short index form for passes that do not cross a multiple of
    // 2^32 (a uniform branch: at most one in 2^20 takes the other);
    // the binary32 commits are bound by HBM, not by VALU issue, and keep
    // the plain form (the short one measured 0.3% slower there, with one
    // more wave per SIMD resident).
    if (kWords16<M> && IndexLo16::applies(a.goff + e0, kPass)) {
        return do_tile_vec<M, IndexLo16, Vec, Rows, false>(a, e0, 0, sc);
    }
    if (!kCommits<M> && same_high_half(a.goff + e0, kPass)) {
        return do_tile_vec<M, IndexHi32, Vec, Rows, false>(a, e0, 0, sc);
    }
    return do_tile_vec<M, IndexAny, Vec, Rows, false>(a, e0, 0, sc);
}
template <Mode M, int Vec>
__device__ __forceinline__ uint64_t do_row(const Arrays& a, uint64_t e0, uint32_t nvec, const StepScalars& sc) {
    return do_tile_vec<M, IndexAny, Vec, 1, true>(a, e0, nvec, sc);
}

// ---------------------------------------------------------------------------
// One workgroup per tile.  The tile's segment comes from the batch's tables
// (kernel arguments, scalar loads); the tile's digest share is summed over the
// workgroup in LDS and handed in with a 64-bit atomic for each of two words.
// ---------------------------------------------------------------------------
template <Mode M, Form F>
__device__ __forceinline__ uint32_t tile_of_block(uint32_t tiles) {
    constexpr Runs kRuns = runs_of(M, F);
    if (tiles >= kRuns.long_from) return dealt_tile(blockIdx.x, tiles, kRuns.long_run);
    if (tiles >= kRuns.from) return dealt_tile(blockIdx.x, tiles, kRuns.run);
    return blockIdx.x;
}

// Has the compiler load what a workgroup needs of the arguments here, in one go:
// it would rather load each where it is used, and the workgroup wait each time.
__device__ __forceinline__ void load_now(Segment& s) {
    asm volatile(""
                 : "+s"(s.elem_begin), "+s"(s.elem_count), "+s"(s.tile_begin), "+s"(s.tile_end), "+s"(s.align),
                   "+s"(s.sc.beta1), "+s"(s.sc.beta2), "+s"(s.sc.eps), "+s"(s.sc.decay), "+s"(s.sc.omb1),
                   "+s"(s.sc.omb2), "+s"(s.sc.step_size), "+s"(s.sc.rs_bc2));
}
__device__ __forceinline__ void load_now(const Arrays& a) {
    asm volatile("" ::"s"(a.p), "s"(a.g), "s"(a.m), "s"(a.v), "s"(a.b), "s"(a.goff));
}
__device__ __forceinline__ void load_now(const ArraysBf16& a) {
    asm volatile("" ::"s"(a.p), "s"(a.g), "s"(a.m), "s"(a.v), "s"(a.goff));
}

template <Mode M, Form F, typename A>
__device__ __forceinline__ void tile_body(const A& a, const Batch& bt, uint64_t* lds) {
    constexpr Shape kShape = shape_of(M, F);
    constexpr int kVecs = kShape.vec, kRows = kShape.rows;
    constexpr uint32_t kPass = kShape.elems();
    const uint32_t passes = kManyPasses<M, F> ? bt.passes : 1;
    const uint32_t tile_elems = kPass * passes;
    // The tile's segment.  Segment 0's line is loaded together with the number of
    // segments, so what a flat shard needs is there after one wait; else the segment
    // is counted out from all tile_begin at once (a binary search waits five times,
    // each time for memory in the first workgroups of a launch).  Against such a search
    // over a table per field: commit of 0.1M and 1M elements 4.95 -> 4.65 and 8.0 -> 7.6 us,
    // guard of 1M 4.5 -> 4.0, commit of 143M in 291 segments 737 -> 732.
    Segment sg = bt.seg[0];
    uint32_t seg = 0, nseg = bt.nseg, tiles = bt.tiles;
    load_now(a);
    asm volatile("" : "+s"(nseg), "+s"(tiles));
    load_now(sg);
    const uint32_t tile = tile_of_block<M, F>(tiles);
    if (nseg > 1) {
#pragma unroll
        for (int k = 1; k < kSegsPerLaunch; ++k) {
            // (two scalar instructions; the compiler takes five and goes through VGPRs)
            asm("s_cmp_ge_u32 %1, %2\n\ts_addc_u32 %0, %0, 0" : "+s"(seg) : "s"(tile), "s"(bt.tile_begin[k]) : "scc");
        }
        sg = bt.seg[seg];
        load_now(sg);
    }
    const StepScalars& sc = sg.sc;
    const uint64_t seg_first = sg.elem_begin;
    const uint64_t seg_end = seg_first + sg.elem_count;
    const uint32_t align = sg.align;
    const uint64_t e0 = seg_first + (align == kNeverAligned ? 0 : align) + (tile - sg.tile_begin) * (uint64_t)tile_elems;
    // This wave's word of the workgroup sum starts at zero (LDS operations of
    // one wave are carried out in the order it issues them, so the clearing
    // comes before the wave's own additions below).
    uint64_t* const wave_sum = lds + (threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0) {
        __hip_atomic_store(wave_sum, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    uint64_t acc = 0;
    if constexpr (kWholeApart<M, F>) {
        const uint64_t left = e0 < seg_end ? seg_end - e0 : 0;
        uint32_t whole = left < tile_elems ? (uint32_t)left / kPass : passes;  // the tile's whole passes
        if (align == kNeverAligned) whole = 0;
        auto one_pass = [&](uint64_t at) { acc += do_pass<M, kVecs, kRows>(a, at, sc); };
        if constexpr (kManyPasses<M, F>) {
#pragma unroll 1
            for (uint32_t pass = 0; pass < whole; ++pass) one_pass(uniform(e0 + pass * kPass));
        } else if (whole != 0) {
            one_pass(e0);
        }
        if (whole < passes || (align != 0 && tile == sg.tile_begin)) {
            // As below.
            uint64_t e, e_end;
            if (align == kNeverAligned) {
                e = e0 + threadIdx.x;
                e_end = (e0 + tile_elems < seg_end) ? e0 + tile_elems : seg_end;
            } else {
                e = e_end = 0;
                const uint64_t at = e0 + whole * kPass;
                if (whole < passes && at < seg_end) {
                    const uint32_t nvec = (uint32_t)(seg_end - at) / kVecs;
#pragma unroll 1
                    for (uint32_t done = 0; done < nvec; done += kBlock) {
                        acc += do_row<M, kVecs>(a, at + done * kVecs, nvec - done, sc);
                    }
                    e = at + nvec * kVecs + threadIdx.x;
                    e_end = seg_end;
                }
                if (tile == sg.tile_begin && threadIdx.x >= 64) {
                    e = seg_first + threadIdx.x - 64;
                    e_end = seg_first + align < seg_end ? seg_first + align : seg_end;
                }
            }
#pragma unroll 1
            for (; e < e_end; e += kBlock) {
                acc += do_scalar<M>(a, e, sc);
            }
        }
    } else {
        // What the tile has for the element-wise path: elements e, e + kBlock, ...
        // below e_end.
        uint64_t e = 0, e_end = 0;
        if (align == kNeverAligned) {
            e = e0 + threadIdx.x;
            e_end = (e0 + tile_elems < seg_end) ? e0 + tile_elems : seg_end;
        } else {
            const uint64_t left = e0 < seg_end ? seg_end - e0 : 0;
            const uint32_t whole = left < tile_elems ? (uint32_t)left / kPass : passes;  // the tile's whole passes
            auto one_pass = [&](uint64_t at) { acc += do_pass<M, kVecs, kRows>(a, at, sc); };
            if constexpr (kManyPasses<M, F>) {
#pragma unroll 1
                for (uint32_t pass = 0; pass < whole; ++pass) one_pass(uniform(e0 + pass * kPass));
            } else if (whole != 0) {
                one_pass(e0);
            }
            const uint64_t at = e0 + whole * kPass;
            if (whole < passes && at < seg_end) {
                // The last pass of a segment: whole vectors, row by row, then the
                // elements behind them.  (With every unaligned segment and every
                // last tile element by element a rank's 20M-element slice of an
                // unpadded vector took 156 us per zeroing commit and 76 + 44 us per
                // BF16 commit and digest, against 125 and 58 + 34 us.)
                const uint32_t nvec = (uint32_t)(seg_end - at) / kVecs;
#pragma unroll 1
                for (uint32_t done = 0; done < nvec; done += kBlock) {
                    acc += do_row<M, kVecs>(a, at + done * kVecs, nvec - done, sc);
                }
                e = at + nvec * kVecs + threadIdx.x;
                e_end = seg_end;
            }
            if (tile == sg.tile_begin && threadIdx.x >= 64) {
                // The first tile's second wave: the elements before the first
                // aligned one (the segment may end among them).
                e = seg_first + threadIdx.x - 64;
                e_end = seg_first + align < seg_end ? seg_first + align : seg_end;
            }
        }
#pragma unroll 1
        for (; e < e_end; e += kBlock) {
            acc += do_scalar<M>(a, e, sc);
        }
    }
    // Workgroup sum: every lane adds its share into its wave's LDS word with
    // one 64-bit LDS atomic (no VALU work: a shuffle tree costs about fifty
    // VALU instructions per lane, a few percent of a digesting kernel), then
    // the threads that hand it in add the four words.
    __hip_atomic_fetch_add(wave_sum, acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    const uint32_t slot = bt.per_segment ? bt.slot0 + seg : 0;
    const uint32_t in_seg = tile - sg.tile_begin;
    // wave 0 for the slot, wave 1 for the total, whose nodes sit beside slot 0's
    const uint32_t wave = uniform(threadIdx.x >> 6);
    const bool total = wave == 1;
    if (wave == 0 || (total && a.res.total_tiles != 0)) {
        uint64_t s = 0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
            s += lds[w];
        }
        if (a.res.words == nullptr) {
            if (threadIdx.x == 0 && s != 0) {
                atomicAdd(reinterpret_cast<unsigned long long*>(a.res.digest + slot), (unsigned long long)s);
            }
        } else if ((threadIdx.x & 63) < 2) {
            const uint32_t n = sg.tile_end - sg.tile_begin;
            uint64_t* const line0 = a.res.words + a.res.set * 2;
            uint64_t* const line = line0 + (uint64_t)slot * kLanes * kLaneStride;
            hand_in(total ? line0 + 8 : line, total ? line0 + kLaneStride + 4 : line + 4,
                    a.res.digest + (total ? a.res.total_slot : slot), total ? a.res.total_tiles : n,
                    total ? bt.tile0 + tile : in_seg, s);
        }
    }
    if (a.res.words != nullptr && in_seg == 0) {
        clear_other_set(a.res, slot);
    }
}

// Waves per SIMD a kernel must be able to keep resident (caps its VGPRs).
// The two standalone digests are bound by VALU issue and keep the full
// eight waves per SIMD (the short index form would otherwise take the state
// digest to 66 VGPRs and seven waves).  The BF16-state commit takes 39 VGPRs in its
// small shape and 64 in the usual one, scheduled for eight waves in the former (6M
// elements 18.6 us against 19.6) and for six in the latter (453M 1115 us against 1128).
template <Mode M, Form F>
constexpr unsigned kMinWavesPerSimd = (M == Mode::StateDigest || M == Mode::DigestBf16State) ? 8u
                                      : (M == Mode::CommitBf16State)                         ? (F == Form::Small ? 8u : 6u)
                                                                                             : 1u;

template <Mode M, Form F>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kMinWavesPerSimd<M, F>)))
void tile_kernel(Arrays a, Batch bt) {
    __shared__ uint64_t lds[kBlock / 64];
    tile_body<M, F>(a, bt, lds);
}

template <Mode M, Form F>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kMinWavesPerSimd<M, F>)))
void tile_kernel_bf16(ArraysBf16 a, Batch bt) {
    __shared__ uint64_t lds[kBlock / 64];
    tile_body<M, F>(a, bt, lds);
}

// Clears what the tile kernels hand their shares in to: every node of both
// sets of the workspace when there is one, else the nslots result slots.
__global__ __launch_bounds__(kBlock) void clear_kernel(uint64_t* digest, uint64_t* words, uint32_t nres,
                                                       uint32_t nslots) {
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    const uint64_t at = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (words) {
        const uint64_t n = (uint64_t)nres * kLanes * kNodesPerLane;
        for (uint64_t i = at; i < n; i += stride) {
            uint64_t* node = words + (i / kNodesPerLane) * kLaneStride + (i % kNodesPerLane) * 2;
            node[0] = 0;
            node[1] = 0;
        }
    } else {
        for (uint64_t i = at; i < nslots; i += stride) {
            digest[i] = 0;
        }
    }
}

// digest[nres] = sum of digest[0..nres): the total of per-segment results
// where the tile kernels do not form it (no workspace, or more segments than
// a node counts).
__global__ __launch_bounds__(kBlock) void total_kernel(uint64_t* digest, uint32_t nres) {
    __shared__ uint64_t lds[kBlock / 64];
    uint64_t total = 0;
    for (uint32_t r = threadIdx.x; r < nres; r += kBlock) {
        total += digest[r];
    }
    const uint64_t t = block_sum(total, lds);
    if (threadIdx.x == 0) {
        digest[nres] = t;
    }
}

// 30 bytes per element with no arithmetic beyond one add, through the commit's
// instructions in tiles of 16 KB per array in plain order: a fixed reference for
// the commit's bytes (whose smaller tiles, with less in flight, may beat it where the
// arrays lie close together).  The outputs may alias the inputs element for element (in
// place).  n is a multiple of 4; the last tile's resources end at n, and a
// vector beyond it is dropped by the buffer range check.
__device__ __forceinline__ void probe_tile(const float* i0, const float* i1, const float* i2, const float* i3,
                                           float* o0, float* o2, float* o3, uint16_t* oh, uint64_t n,
                                           uint64_t tile) {
    constexpr uint32_t kRow32 = kBlock * kVec * 4;
    constexpr uint32_t kRow16 = kBlock * kVec * 2;
    const uint64_t e0 = tile * kTile;
    const uint64_t left = n - e0;
    const uint32_t cnt = left < (uint64_t)kTile ? (uint32_t)left : (uint32_t)kTile;
    const auto r0 = tile_rsrc(i0 + e0, cnt * 4), r1 = tile_rsrc(i1 + e0, cnt * 4);
    const auto r2 = tile_rsrc(i2 + e0, cnt * 4), r3 = tile_rsrc(i3 + e0, cnt * 4);
    const auto w0 = tile_rsrc(o0 + e0, cnt * 4), w2 = tile_rsrc(o2 + e0, cnt * 4);
    const auto w3 = tile_rsrc(o3 + e0, cnt * 4), wh = tile_rsrc(oh + e0, cnt * 2);
    const uint32_t lane32 = threadIdx.x * kVec * 4, lane16 = threadIdx.x * kVec * 2;
    u32x4 A[kUnroll], B[kUnroll], C[kUnroll], D[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        A[u] = load16(r0, lane32 + u * kRow32);
        B[u] = load16(r1, lane32 + u * kRow32);
        C[u] = load16(r2, lane32 + u * kRow32);
        D[u] = load16(r3, lane32 + u * kRow32);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        u32x4 s;
#pragma unroll
        for (int j = 0; j < kVec; ++j) {
            s[j] = __float_as_uint(__uint_as_float(A[u][j]) + __uint_as_float(B[u][j]));
        }
        store16(s, w0, lane32 + u * kRow32);
        store16(C[u], w2, lane32 + u * kRow32);
        store16(D[u], w3, lane32 + u * kRow32);
        u32x2 h;
        h.x = (s.x >> 16) | (s.y & 0xFFFF0000u);
        h.y = (s.z >> 16) | (s.w & 0xFFFF0000u);
        store8(h, wh, lane16 + u * kRow16);
    }
}

// One workgroup per tile.
__global__ __launch_bounds__(kBlock) void probe_kernel(const float* i0, const float* i1, const float* i2,
                                                       const float* i3, float* o0, float* o2, float* o3,
                                                       uint16_t* oh, uint64_t n) {
    probe_tile(i0, i1, i2, i3, o0, o2, o3, oh, n, blockIdx.x);
}

// The same work from a persistent grid: workgroup b takes tiles b, b + grid,
// b + 2 grid, ... (the grid-stride shape), for comparison with one
// workgroup per tile.
__global__ __launch_bounds__(kBlock) void probe_persistent_kernel(const float* i0, const float* i1,
                                                                  const float* i2, const float* i3, float* o0,
                                                                  float* o2, float* o3, uint16_t* oh, uint64_t n) {
    const uint64_t tiles = (n + kTile - 1) / kTile;
    for (uint64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        probe_tile(i0, i1, i2, i3, o0, o2, o3, oh, n, t);
    }
}

}  // namespace

hipError_t launch_clear(uint64_t* digest, uint64_t* words, uint32_t nres, uint32_t nslots, hipStream_t stream) {
    const uint64_t n = words ? (uint64_t)nres * kLanes * kNodesPerLane : nslots;
    const uint32_t grid = (uint32_t)std::min<uint64_t>((n + kBlock - 1) / kBlock, 1024);
    hipLaunchKernelGGL(clear_kernel, dim3(grid), dim3(kBlock), 0, stream, digest, words, nres, nslots);
    return hipGetLastError();
}

namespace {

// LDS reserved per workgroup beyond what it uses: holds the binary32 commits
// at five workgroups per CU.
//
// A commit reads four arrays and writes four, and HBM gives such a mix its
// reading rate only while few rows are open: what counts is how much of each
// array is in flight at a time, and in what order.  Tiles of 16 KB per array, as
// many as fit (four per CU), kept 16 MB of each in flight; tiles of 4 KB, five per
// CU, keep 5 MB, and runs of neighbouring tiles per XCD keep that in a few
// stretches.  One commit of 453,001,472 elements, the arrays in five separate
// allocations, us (TB/s), and in an arena (arrays 44 GiB apart):
//   16 KB tiles, four per CU               2420 (5.62)   2095
//   4 KB tiles, eight per CU               2360 (5.76)   2101
//   4 KB tiles, five per CU                2272 (5.98)   2105
//   4 KB tiles, eight per CU, runs of 32   2251 (6.04)   2092
//   4 KB tiles, five per CU, runs of 32    2205 (6.16)   2078
//   4 KB tiles, four per CU, runs of 32    2170 (6.26)   2117
//   4 KB tiles, three per CU               2721 (4.99)
// Five rather than four keeps the arena's rate.  The 16-bit state's commit and
// the digests were slower with less in flight.
template <Mode M, Form F>
constexpr uint32_t kReserveLds = kCommits<M> && F == Form::Usual ? 30u << 10 : 0u;

template <Mode M>
void launch_tiles(Form form, const Arrays& a, const Batch& b, uint32_t grid, hipStream_t stream) {
    auto launch = [&](auto kernel, uint32_t lds) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), lds, stream, a, b);
    };
    if constexpr (small_up_to(M) != 0) {
        if (form == Form::Small) return launch(tile_kernel<M, Form::Small>, 0);
    }
    if constexpr (has_long(M)) {
        if (form == Form::Long) return launch(tile_kernel<M, Form::Long>, kReserveLds<M, Form::Long>);
    }
    launch(tile_kernel<M, Form::Usual>, kReserveLds<M, Form::Usual>);
}

template <Mode M>
void launch_tiles(Form form, const ArraysBf16& a, const Batch& b, uint32_t grid, hipStream_t stream) {
    if (form == Form::Small) {
        hipLaunchKernelGGL((tile_kernel_bf16<M, Form::Small>), dim3(grid), dim3(kBlock), 0, stream, a, b);
    } else {
        hipLaunchKernelGGL((tile_kernel_bf16<M, Form::Usual>), dim3(grid), dim3(kBlock), 0, stream, a, b);
    }
}

}  // namespace

hipError_t launch_batch(Mode mode, Form form, const Arrays& a, const Batch& b, uint32_t grid, hipStream_t stream) {
    switch (mode) {
        case Mode::Commit: launch_tiles<Mode::Commit>(form, a, b, grid, stream); break;
        case Mode::StateDigest: launch_tiles<Mode::StateDigest>(form, a, b, grid, stream); break;
        case Mode::Bf16Digest: launch_tiles<Mode::Bf16Digest>(form, a, b, grid, stream); break;
        case Mode::CommitZeroGrad: launch_tiles<Mode::CommitZeroGrad>(form, a, b, grid, stream); break;
        case Mode::GradGuard: launch_tiles<Mode::GradGuard>(form, a, b, grid, stream); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_batch_bf16(Mode mode, Form form, const ArraysBf16& a, const Batch& b, uint32_t grid,
                             hipStream_t stream) {
    switch (mode) {
        case Mode::CommitBf16State: launch_tiles<Mode::CommitBf16State>(form, a, b, grid, stream); break;
        case Mode::DigestBf16State: launch_tiles<Mode::DigestBf16State>(form, a, b, grid, stream); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_total(uint64_t* digest, uint32_t nres, hipStream_t stream) {
    hipLaunchKernelGGL(total_kernel, dim3(1), dim3(kBlock), 0, stream, digest, nres);
    return hipGetLastError();
}

hipError_t launch_probe(const float* i0, const float* i1, const float* i2, const float* i3,
                        float* o0, float* o2, float* o3, uint16_t* oh, uint64_t n, uint32_t workgroups,
                        hipStream_t stream) {
    if (workgroups == 0) {
        const uint64_t tiles = (n + kTile - 1) / kTile;
        hipLaunchKernelGGL(probe_kernel, dim3((uint32_t)tiles), dim3(kBlock), 0, stream, i0, i1, i2, i3, o0, o2,
                           o3, oh, n);
    } else {
        hipLaunchKernelGGL(probe_persistent_kernel, dim3(workgroups), dim3(kBlock), 0, stream, i0, i1, i2, i3, o0,
                           o2, o3, oh, n);
    }
    return hipGetLastError();
}

}  // namespace pact
