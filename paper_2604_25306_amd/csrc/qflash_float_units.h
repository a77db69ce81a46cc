// The steps of the integer algorithm that the kernels do on the single-precision units, or on accumulators and scores
// that carry an offset, and the constants they stand on.  No HIP in it: tests/test_float_units.py compiles this file for
// the host and enumerates every identity with real floats, rounded down as the kernels round (round_down in qflash_tile.h).
#pragma once
#include <stdint.h>

#include "qflash_internal.h"

#if defined(__FAST_MATH__) || __FINITE_MATH_ONLY__
#error "every float operation here is meant exactly as written, denormals and the sign of zero included"
#endif

namespace {

QF_UNIT_HD inline float qf_as_float(uint32_t bits) { return __builtin_bit_cast(float, bits); }
QF_UNIT_HD inline uint32_t qf_as_bits(float f) { return __builtin_bit_cast(uint32_t, f); }
QF_UNIT_HD inline uint32_t qf_umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }

constexpr int kNegBig = -(1 << 30);   // stands for "excluded": far below any clamp point (so is
                                      // anything a saturating add of INT32_MIN produces)
constexpr int kMInit = -(1 << 21);    // initial running maximum (Algorithm 1)

// ScaleRelease with alpha in 16 fractional bits, floor(x * alpha16 / 2^16), 0 <= alpha16 <= 2^16.
//
// Integer form.  Numerator accumulators are kept with an offset, y = x + 2^30 > 0 (the MFMA adds products modulo
// 2^32, so the offset rides along).  With A = alpha16 << 16:
//   mul_hi_u32(y, A) = floor((x A + 2^30 A) / 2^32) = floor(x alpha16 / 2^16) + A/4   (A is a multiple of 4)
// so the rescaled accumulator, again offset by 2^30, is mul_hi_u32(y, A) + (2^30 - A/4): one
// multiply-high and one add, no shift.  alpha16 = 2^16 (identity) does not fit A; there
// A = 2^32 - 1 gives mul_hi_u32(y, A) = y - 1 for every 1 <= y < 2^32, and the addend is 1.
// (|x| < 2^26 always.)  The offset is 2^30 because that bit pattern (the float 2.0) is an inline
// constant of the instruction set: a matrix instruction can start from a block of it without a
// single register being set aside for it.
constexpr int kAccBias = 0x40000000;   // offset carried by biased scores, and by the numerator accumulators of QMAX
struct ReleaseConst {
    unsigned A, C;       // accumulator: y <- mul_hi_u32(y, A) + C
    int alpha14;         // alpha16 << 14, for the (unbiased, non-negative) denominator
};
QF_UNIT_HD inline ReleaseConst make_release(unsigned alpha16) {
    ReleaseConst r;
    const unsigned one = alpha16 >> 16;   // 1 only for the identity
    r.A = (alpha16 << 16) - one;
    r.C = (unsigned)kAccBias - (alpha16 << 14) + one;
    r.alpha14 = (int)(alpha16 << 14);
    return r;
}
QF_UNIT_HD inline int release_acc(int y, const ReleaseConst& r) { return (int)(qf_umulhi((unsigned)y, r.A) + r.C); }
// Denominator: 0 <= l < 2^20, floor(l * alpha16 / 2^16) = ((l << 2) * (alpha16 << 14)) >> 32.
QF_UNIT_HD inline int release_l(int l, const ReleaseConst& r) { return (int)(((int64_t)(l << 2) * r.alpha14) >> 32); }

// The same for accumulators offset by 2^23 (kAccOffset), in one instruction: seen as a float, an integer below
// 2^24 is that many units of 2^-149, denormal or not, so that a fused multiply-add that rounds toward minus
// infinity (round_down) is floor(x alpha16 / 2^16) + 2^23, y = x + 2^23, with the addend 2^23 - 2^7 alpha16, as
// long as -2^23 <= x < 2^23.  |x| <= 128 l + 129 per tile, so l < 65000 (kFloatReleaseMaxL) keeps it there; always
// where N <= 256.  Beyond it the integer form above takes over, between two changes of offset.
//
// Why floats: of the vector units of a SIMD, one instruction in four cycles is all that integer work gets
// (4.1 cycles measured with four wavefronts for any mix of multiplies, maxima, permutes, subtractions), but
// fused multiply-adds issue beside it (2.2 to 2.4 cycles per instruction for a mix of half and half).  A
// v_dot4 or a 24-bit multiply among them stops that for some forty instructions (4.1 cycles with one in
// sixteen), which is why neither is used in the loop over the tiles.
constexpr int kAccOffset = 1 << 23;
constexpr int kFloatReleaseMaxL = 65000;
struct FloatRelease { float alpha, add; };
QF_UNIT_HD inline FloatRelease make_float_release(unsigned alpha16) {
    return FloatRelease{(float)alpha16 * 0x1p-16f, qf_as_float((uint32_t)(kAccOffset - (int)(alpha16 << 7)))};
}
QF_UNIT_HD inline int release_acc(int y, const FloatRelease& r) {
    return (int)qf_as_bits(__builtin_fmaf(qf_as_float((uint32_t)y), r.alpha, r.add));
}
QF_UNIT_HD inline int release_l(int l, const FloatRelease& r) { return (int)qf_as_bits(qf_as_float((uint32_t)l) * r.alpha); }

// Four weights below 128, one to a register, to the bytes of one: the first three as floats (integers below 2^24,
// exact in any rounding), see above.
QF_UNIT_HD inline unsigned pack_weights(unsigned p0, unsigned p1, unsigned p2, unsigned p3) {
    const float w = __builtin_fmaf(__builtin_fmaf(qf_as_float(p2), 256.0f, qf_as_float(p1)), 256.0f, qf_as_float(p0));
    return (p3 << 24) | qf_as_bits(w);
}

// Offset of the biased scores of 32-key block kb of a tile, relative to kAccBias.  A matrix
// instruction takes a constant as its addend only if the constant is one of the few the instruction
// set has built in (here the bit patterns of 1 / (2 pi), 2.0, 4.0 and 1.0) and, with this compiler, only if no other
// instruction shares it; a block of sixteen registers filled with the constant costs eight vector and
// sixteen scalar instructions per tile otherwise.  So each block of a tile gets a constant of its own, and the
// two places that compare scores across blocks (the row maximum, the table index) take the difference out again.
// Block 0 has the only one of them around which 2^21 integers either way lie in one binade, [1/8, 1/4): its scores
// are floats 2^-26 apart, and a fused multiply-add makes the table index of them (float_index).
constexpr int kScoreOffset0 = 0x3E22F983;
QF_UNIT_HD constexpr int score_offset_delta(int kb) {
    return kb == 0 ? kScoreOffset0 - kAccBias : kb == 1 ? 0 : kb == 2 ? (1 << 23) : -(1 << 23);
}
// A key beyond the sequence, as a biased score at the common offset: below every real score and every table edge
// (which are at least -2^21 - 40960), and still in the binade of block 0.
constexpr int kMaskedBiased = kAccBias - (kScoreOffset0 - 0x3E000000);
// max(0, s - edge) for a score s of block 0 and the edge -- the score of table index 0 -- at the common offset:
// s 2^-123 is s - 0x3E000000 + 2^23 units of 2^-149, and so is the addend; the clamp to [0, 1] is the maximum.
constexpr uint32_t kIndexScale = 0x02000000;   // 2^-123
QF_UNIT_HD inline float index_addend(unsigned edge) {
    return qf_as_float(edge + ((unsigned)score_offset_delta(0) - 0x3E000000u + 0x800000u + 0x80000000u));
}
QF_UNIT_HD inline unsigned float_index(int s, float scale /* kIndexScale */, float addend) {
    const float i = __builtin_fmaf(qf_as_float((uint32_t)s), scale, addend);
#if defined(__HIP_DEVICE_COMPILE__)
    return qf_as_bits(__builtin_amdgcn_fmed3f(i, 0.0f, 1.0f));
#else
    return qf_as_bits(i > 0.0f ? (i < 1.0f ? i : 1.0f) : 0.0f);
#endif
}

// Normalisation with floats, floor(x / l) + 128 before the saturation to a byte, for l <= kFloatNormaliseMaxL:
// (x + 1/2) R + 128 rounded down, with R = v_rcp(l).  (x + 1/2) / l is at least 1 / (2 l) from any integer, and where it
// matters, |x / l| <= 128, off by 128 2^-23 at most if v_rcp is off by one unit in the last place at most, which is what
// the instruction promises: less than 1 / (2 l) for l < 32768.  The limit is the largest l of 256 keys.
// OFFSET kAccOffset: y = x + 2^23 as a float is (x + 2^23) 2^-149, so y 2^126 - (1 - 2^-24) is (x + 1/2) 2^-23.
// OFFSET kScoreOffset0 (one KV tile of at most 64 keys: |x| < 2^20, l <= 8128): y is (x + 10680707) 2^-26 and the half goes
// to the addend, 128 + 1 / (2 l) rounded down to a multiple of 2^-16: both errors together stay below 1 / (2 l).
constexpr int kFloatNormaliseMaxL = 127 * 256;
template <int OFFSET>
struct FloatQuotient {
    static_assert(OFFSET == kAccOffset || OFFSET == kScoreOffset0, "the offsets whose bits are evenly spaced floats");
    float R, c;
    QF_UNIT_HD explicit FloatQuotient(float r /* 1 / l; 0 where there is no key: 128 -> output 0 */)
        : R(r * 0x1p23f), c(OFFSET == kAccOffset ? 128.0f : __builtin_fmaf(r, 0.5f, 128.0f)) {}
    static constexpr uint32_t kScale = OFFSET == kAccOffset ? 0x7e800000u /* 2^126 */ : 0x41000000u /* 8 */;
    QF_UNIT_HD float operator()(int y, float scale) const {
        constexpr float base = OFFSET == kAccOffset ? -1.0f + 0x1p-24f : -10680707.0f * 0x1p-23f;
        return __builtin_fmaf(__builtin_fmaf(qf_as_float((uint32_t)y), scale, base), R, c);
    }
};

}  // namespace
