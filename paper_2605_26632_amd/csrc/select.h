// Device helpers of the online 2:4 sparsification, shared by the sweeps that perform it: magnitude
// Top-2 of an aligned group of four (Alg. 1 "X~ <- TopK(X)"), the norm-compensation factor of the
// method section ("Norm-Compensated Sparsification", s = sqrt(|X|^2 / (|X~|^2 + eps))) and the E4M3
// conversion of the FP8 composition.
#pragma once
#include "rtl_internal.h"

namespace rtl {

__device__ __forceinline__ float bits_to_f32(uint32_t u) { return __uint_as_float(u); }

// fp32 -> bf16 round-to-nearest-even, NaN kept (quiet bit set).
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    uint32_t nan = (u >> 16) | 0x40u;
    return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? nan : r;
}

struct GroupOut {
    uint32_t packed;  // two kept bf16: lower position in the low half
    uint32_t nibble;  // pos0 | pos1 << 2
    float num, den;   // sum of squares of the four / of the two kept
};

// Two fp32 values -> two E4M3 codes (low byte = first): round to nearest even, saturating at
// +-448 (so do +-inf), NaN -> 0x7F. The hardware conversion is exact for |t| <= 448 but turns
// larger magnitudes into NaN codes, hence the clamp.
__device__ __forceinline__ uint32_t e4m3_pair(float t0, float t1) {
    const float c0 = __builtin_amdgcn_fmed3f(t0, -448.f, 448.f);
    const float c1 = __builtin_amdgcn_fmed3f(t1, -448.f, 448.f);
    uint32_t p = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c0, c1, 0, false) & 0xFFFFu;
    if (__builtin_isunordered(t0, t1)) {   // rare: at least one NaN
        if (t0 != t0) p = (p & 0xFF00u) | 0x7Fu;
        if (t1 != t1) p = (p & 0x00FFu) | 0x7F00u;
    }
    return p;
}

// The compensation factor exactly as defined: every square rounded on its own, the sums in the
// stated order, IEEE divide and square root. Squares of bf16 values are exact in fp32 unless they
// fall below 2^-126, so the fused multiply-adds of the fast path give the same sums for ordinary
// magnitudes; for tiny ones (|x| < 2^-63) only this unfused form matches a plain evaluation.
__device__ __forceinline__ float exact_group_scale(uint32_t d0, uint32_t d1, float ka, float kb, float eps) {
#pragma clang fp contract(off)
    const float f0 = bits_to_f32(d0 << 16), f1 = bits_to_f32(d0 & 0xFFFF0000u);
    const float f2 = bits_to_f32(d1 << 16), f3 = bits_to_f32(d1 & 0xFFFF0000u);
    const float q0 = f0 * f0, q1 = f1 * f1, q2 = f2 * f2, q3 = f3 * f3;
    const float num = ((q0 + q1) + q2) + q3;
    const float qa = ka * ka, qb = kb * kb;
    const float den = (qa + qb) + eps;
    return sqrtf(num / den);
}

typedef short i16x2 __attribute__((ext_vector_type(2)));

// acc + x_lo^2 + x_hi^2 of a packed bf16 pair, one instruction.
__device__ __forceinline__ float dot2_bf16(uint32_t x, float acc) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v = __builtin_bit_cast(bf16x2, x);
    return __builtin_amdgcn_fdot2_f32_bf16(v, v, acc, false);
}

// d0 = x0 | x1 << 16, d1 = x2 | x3 << 16 (bf16 bit patterns). With FP8 the kept pair leaves as two
// E4M3 codes of (s * x) * inv (inv = 1 / x_scale) in the low 16 bits of `packed`.
template <int COMP, bool FP8 = false>
__device__ __forceinline__ GroupOut select_group(uint32_t d0, uint32_t d1, float eps, float inv = 1.0f) {
    // Top-2 on packed 15-bit magnitudes, positions (0, 2) in one register and (1, 3) in the other, so that one
    // packed instruction serves both pairs (0, 1) and (2, 3). The kept set is one of three: both of the first
    // pair (its loser is no smaller than the second pair's winner: the lower index wins a tie), both of the
    // second (its loser is larger than the first pair's winner), else the winners of the two pairs.
    const uint32_t even = __builtin_amdgcn_perm(d1, d0, 0x05040100u), odd = __builtin_amdgcn_perm(d1, d0, 0x07060302u);
    const i16x2 me = __builtin_bit_cast(i16x2, even & 0x7FFF7FFFu), mo = __builtin_bit_cast(i16x2, odd & 0x7FFF7FFFu);
    const i16x2 hi = __builtin_elementwise_max(me, mo), lo = __builtin_elementwise_min(me, mo);   // .x: pair (0, 1), .y: pair (2, 3)
    const i16x2 odd_wins = (me - mo) >> 15;                  // all ones where the odd position is strictly larger
    uint32_t mask = __builtin_bit_cast(uint32_t, odd_wins);
    asm("" : "+v"(mask));                                    // (keeps the select below one bit-field insert)
    const bool both01 = lo.x >= hi.y, both23 = lo.y > hi.x;
    const uint32_t winners = (mask & odd) | (~mask & even);
    const uint32_t pair = both01 ? d0 : (both23 ? d1 : winners);
    // winners' nibble: pos0 = 0 or 1, pos1 = 2 or 3 -> 8 + (1 wins over 0) + 4 (3 wins over 2)
    const uint32_t winners_nibble = (uint32_t)__builtin_amdgcn_sdot2(__builtin_bit_cast(i16x2, mask), i16x2{-1, -4}, 8, false);
    GroupOut o;
    o.nibble = both01 ? 0x4u : (both23 ? 0xEu : winners_nibble);
    o.num = 0.f;
    o.den = 0.f;
    if constexpr (COMP == RTL_COMP_ROW || COMP == RTL_COMP_TENSOR) {
        const float f0 = bits_to_f32(d0 << 16), f1 = bits_to_f32(d0 & 0xFFFF0000u);
        const float f2 = bits_to_f32(d1 << 16), f3 = bits_to_f32(d1 & 0xFFFF0000u);
        const float ka = bits_to_f32(pair << 16), kb = bits_to_f32(pair & 0xFFFF0000u);
        // squares of bf16 values are exact in fp32; the additions are in the stated order
        // (fused multiply-adds round exactly like a multiply and an add here, see exact_group_scale)
        o.num = __builtin_fmaf(f3, f3, __builtin_fmaf(f2, f2, __builtin_fmaf(f1, f1, f0 * f0)));
        o.den = __builtin_fmaf(kb, kb, ka * ka);
    }
    if constexpr (COMP == RTL_COMP_GROUP) {
        // The stored values are bf16_rne(s * k) with s = sqrtf(num / den) in IEEE fp32. The exact sequence
        // (exact_group_scale) costs ~40 instructions, enough to make this sweep ALU bound, so s is first taken
        // from two-term bf16 dot products, the 1-ulp hardware reciprocal and the square root. Errors in half-units
        // of fp32, relative to the real value: a dot product -3 .. +1 (two addends cut at the end of the largest
        // and one rounding; 4M random pairs: -2.92 .. +1.00), so num -6 .. +2 and den -3 .. +1, reciprocal and
        // product 3: the quotient -10 .. +8, after the root -5 .. +4, the root itself 2, s * k 1: -8 .. +7. The
        // exact sequence: 3 in num, 2 in den, 1 for the quotient, 3 after the root, 1 and 1: 5. The two differ by
        // at most 13; the exact sequence only runs when a fast product lies within 16 units of a bf16 rounding
        // boundary, i.e. whenever they could round differently. The result is bit-identical.
        // The rounding of the dot product is that measurement, not a specification; its model has 3 half-units to spare.
        // Against selection on 17-bit keys with fused multiply-adds for the norms (fast path of the block-mapped kernel, addressing
        // and stores included, 67 vector instructions per group, 51 now; selection and compensation alone 51 and 37): sweep of
        // rtl_sparse_linear back to back [4096, 12288] 30.8 -> 27.6 us (5.7 TB/s), inside calls 35.0 -> 31.8, [4608, 3072] 11.0 -> 10.3,
        // NONE [4096, 12288] 25.9 -> 25.5.
        const float num = dot2_bf16(d1, dot2_bf16(d0, 0.f));
        const float d = dot2_bf16(pair, eps);
        float s = __builtin_amdgcn_sqrtf(num * __builtin_amdgcn_rcpf(d));
        const float ka = bits_to_f32(pair << 16), kb = bits_to_f32(pair & 0xFFFF0000u);
        float p0 = s * ka, p1 = s * kb;
        // tiny (but non-zero) or huge / non-finite scopes are left to the exact sequence too
        const uint32_t nb = __float_as_uint(num);
        const bool odd_range = (nb - 0x0D800000u >= 0x63800000u) & (nb != 0u);
        if constexpr (FP8) {
            // Same idea one rounding later: t = p * inv is what gets rounded, to 3 mantissa
            // bits. The fast and the exact p differ by at most 13 half-units, which the common
            // multiplication by inv and its own rounding turn into at most 15 of t, i.e.
            // less than 2^-20 |t|. The conversion is monotone, so if t (1 - 2^-17) and
            // t (1 + 2^-17), which bracket the exact t even after their own roundings, give the
            // same code, the exact t gives it too, wherever the format's boundaries sit
            // (normal range, subnormal range, saturation: beyond 448 the raw conversion returns
            // the NaN code on both sides, or differs across the limit and the exact sequence runs).
            float t0 = p0 * inv, t1 = p1 * inv;
            constexpr float kBelow = 1.0f - 0x1p-17f, kAbove = 1.0f + 0x1p-17f;
            const uint32_t c_below = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(t0 * kBelow, t1 * kBelow, 0, false);
            const uint32_t c_above = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(t0 * kAbove, t1 * kAbove, 0, false);
            if ((c_below != c_above) | odd_range) {
                s = exact_group_scale(d0, d1, ka, kb, eps);
                t0 = (s * ka) * inv;
                t1 = (s * kb) * inv;
                o.packed = e4m3_pair(t0, t1);
            } else if (fmaxf(fabsf(t0), fabsf(t1)) <= 448.0f) {
                o.packed = c_below & 0xFFFFu;      // inside the format's range the raw conversion is the code
            } else {
                o.packed = e4m3_pair(t0, t1);      // saturating values: the raw conversion returns NaN codes
            }
            return o;
        }
        // low halves in the window [0x8000 - 16, 0x8000 + 16)
        const uint16_t l0 = (uint16_t)(__float_as_uint(p0) + 16u - 0x8000u), l1 = (uint16_t)(__float_as_uint(p1) + 16u - 0x8000u);
        const bool near = (l0 < l1 ? l0 : l1) < 32;
        if (near | odd_range) {
            s = exact_group_scale(d0, d1, ka, kb, eps);
            p0 = s * ka;
            p1 = s * kb;
        }
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const f32x2 pp = {p0, p1};
        const bf16x2 pb = __builtin_convertvector(pp, bf16x2);   // RNE, one instruction on gfx950
        o.packed = __builtin_bit_cast(uint32_t, pb);
        return o;
    }
    if constexpr (FP8) {
        o.packed = e4m3_pair(bits_to_f32(pair << 16) * inv, bits_to_f32(pair & 0xFFFF0000u) * inv);
        return o;
    }
    o.packed = pair;
    return o;
}

}  // namespace rtl
