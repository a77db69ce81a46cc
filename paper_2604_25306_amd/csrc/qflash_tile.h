// Per-tile device code of the integer-only attention forward pass (Algorithm 1, steps 1-11), shared by
// every gfx950 kernel that walks over KV tiles: the operand layout in registers, the element-wise
// integer softmax of one tile, ScaleRelease, the final normalisation.  Included by the kernel
// source files only.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "qflash_internal.h"
#include "qflash_device.h"
#include "qflash_float_units.h"

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v4i_a4 __attribute__((ext_vector_type(4), aligned(4)));

namespace {

// ------------------------------------------------------------------ scalar building blocks

// The two lanes l and l ^ 32 hold the halves of one query row.  One cross-lane swap in the vector
// ALU (no round trip through the LDS crossbar) hands each of them both values: the swap exchanges
// the upper half of its first operand with the lower half of the second, so with both operands
// equal to v every lane ends up with {own, partner's} in some order -- enough for max and sum.
struct HalfPair { int x, y; };
__device__ __forceinline__ HalfPair both_halves(int v) {
    const auto sw = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return HalfPair{(int)sw[0], (int)sw[1]};
}

// Gather byte 3 of four dwords into one dword (v_perm_b32: selector bytes 0-3 pick from the
// second operand, 4-7 from the first).
__device__ __forceinline__ unsigned pack_byte3(unsigned p0, unsigned p1, unsigned p2, unsigned p3) {
    unsigned w = __builtin_amdgcn_perm(p1, p0, 0x07030703u);   // [p0.3, p1.3, .., ..]
    w = __builtin_amdgcn_perm(p2, w, 0x07070100u);             // [p0.3, p1.3, p2.3, ..]
    return __builtin_amdgcn_perm(p3, w, 0x07020100u);          // [p0.3, p1.3, p2.3, p3.3]
}
template <int BYTE>
__device__ __forceinline__ unsigned pack_byte(unsigned p0, unsigned p1, unsigned p2, unsigned p3) {
    constexpr unsigned b = BYTE, h = BYTE + 4;
    unsigned w = __builtin_amdgcn_perm(p1, p0, (h << 24) | (b << 16) | (h << 8) | b);
    w = __builtin_amdgcn_perm(p2, w, (h << 24) | (h << 16) | 0x0100u);
    return __builtin_amdgcn_perm(p3, w, (h << 24) | 0x020100u);
}

// The rest of a kernel behind this call rounds single precision down.  Ahead of it: the scales of a dynamic call, which
// round to nearest, and integer divisions by numbers that may exceed 2^24 (bias_lane_base: heads and bias extents of
// one-token sequences).  The compiler makes a division of v_rcp and products of floats and relies on a first guess that
// is not too large; a divisor cut down to 24 bits makes it larger.  Behind it divisors are small, exact as floats, and
// rounding down only makes the guess smaller, corrected as ever.
// The compiler does not know what the call does.  What keeps arithmetic on its side of it is data: the floats behind it come of
// products of LDS contents read behind a barrier further on, and what has to round to nearest has gone to LDS, or to a scalar
// register by an assembly statement (bias_lane_base), ahead of it.  tests/test_rounding_mode.py reads that from the built code.
__device__ __forceinline__ void round_down() { __builtin_amdgcn_s_setreg(1 | (0 << 6) | (1 << 11), 2); }   // MODE.round, single precision
// Mask of the first n bytes (n <= 0: none, n >= 4: all).
__device__ __forceinline__ unsigned first_bytes(int n) { return (unsigned)(0xffffffffull >> (8 * (4 - min(max(n, 0), 4)))); }
// Sum of the four bytes of w, added to sum.
__device__ __forceinline__ int add_bytes(unsigned w, int sum) { return (int)__builtin_amdgcn_sad_u8(w, 0u, (unsigned)sum); }

// A result block full of the offset (the compiler turns it into the inline constant).
template <int OFFSET = kAccBias>
__device__ __forceinline__ v16i offset_block() {
    v16i z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = OFFSET;
    return z;
}
template <int KBI>
__device__ __forceinline__ v16i score_offset_block() {
    v16i z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = kAccBias + score_offset_delta(KBI);
    return z;
}

// One byte of the weight table.  The table is the first thing in the workgroup's LDS (the resident
// kernel has no other LDS object, so its dynamic LDS starts at address 0): the index is the address.
typedef const __attribute__((address_space(3))) uint8_t lds_u8;
__device__ __forceinline__ int table_weight(unsigned idx) { return (int)*(lds_u8*)(size_t)idx; }

// R = ceil(2^(2L+8) / d) for d in (2^(L-1), 2^L], L = 16 or 20, in integer arithmetic only:
// Newton's iteration for 1/d on 32-bit fixed point (32-bit multiply-high is full rate here),
// then one exact remainder step.  With d31 = d << (31-L) in (2^30, 2^31] and x ~ 2^62 / d31:
//   x0 = (48/17 - 32/17 * d31/2^31) * 2^31,   x <- (x * (2^31 - (d31 * x >> 32)) >> 32) << 2   (3 times)
// q = x >> (23-L) is floor((2^(2L+8) - 1) / d) to within +-1 for every d of both ranges (checked by
// enumerating all of them; tests/test_host_logic.py repeats that); the low 32 bits of the remainder
// (2^(2L+8) - 1) - q d decide the correction, and R = q + 1.
template <int L>
__device__ __forceinline__ unsigned recip_ceil(unsigned d) {
    const unsigned d31 = d << (31 - L);
    unsigned x = (3031741621u - __umulhi(4042322161u, d31)) << 1;
#pragma unroll
    for (int it = 0; it < 3; ++it) {
        const unsigned f = 0x80000000u - __umulhi(d31, x);
        x = __umulhi(x, f) << 2;
    }
    unsigned q = x >> (23 - L);
    const int rem = (int)(0xffffffffu - q * d);
    if (rem < 0) q -= 1;
    else if ((unsigned)rem >= d) q += 1;
    return q + 1;
}

// Quantised-maximum variant: the reference level the initial maximum -2^21 rounds up to,
// ceil(-2^21 / s_inv) * s_inv = -floor(2^21 / s_inv) * s_inv (a_mul = ceil(2^30 / s_inv)).
__device__ __forceinline__ int qmax_initial_reference(int s_inv, int a_mul) {
    unsigned q = __umulhi(1u << 23, (unsigned)a_mul);
    if (q * (unsigned)s_inv > (1u << 21)) q -= 1;
    return -(int)(q * (unsigned)s_inv);
}

// ---------------------------------------------------------------------- per-wavefront state

template <int D>
struct RowState {
    v16i acc[D / 32];   // O^T: features 32*t + 8*(v/4) + 4*g + v%4 of this lane's query row
    int l;              // running denominator
    int m;              // running maximum
};

// What a kernel does ahead of the first read of the tile's V (before_v of process_tile).
struct NothingBeforeV { __device__ __forceinline__ void operator()() const {} };

// One KV tile for one wavefront.  sK: K rows of the tile (row pitch KROW), sV: V^T with the tile's
// columns starting at column 0 (row pitch VROW).  n_valid = number of real kv rows in the tile.
// QMAX selects the quantised-maximum variant, which is NOT Algorithm 1 as printed: RowState::m is
// then the reference level (the running maximum rounded up to a multiple of s_inv; x_shift must be
// 0), scores are referred to it, and ScaleRelease is an exact shift.
// XM selects how the int8 weight of a score is obtained: kExpShift (Algorithm 2 + Eq. 10 in the
// ALUs, any x_shift), kExpShift0 (the same, x_shift == 0) or kExpTable (one LDS look-up in a table
// of the same function, see qflash_build_table).
//
// Offsets.  Numerator accumulators always carry one, which depends on how they are rescaled (kRelease...).  In table mode without
// bias the scores can carry it too (SB): the first MFMA of a score block starts from a
// block of the offset instead of zeros, which costs nothing, and then
//   table index = max(0, s - m + x_p) = (s + 2^30) -sat- (m + 2^30 - x_p)
// is a single unsigned saturating subtraction per score (both operands are positive: |s| < 2^21; block 0: float_index);
// RowState::m holds m + 2^30.  Algorithm 2 for alpha only sees differences, which are unchanged.
enum { kExpShift = 0, kExpShift0 = 1, kExpTable = 2, kExpAuto = 3 };   // kExpAuto: per workgroup, table if its head has one
// Bias of a kernel variant: none, the plain [N,N] layout, or the lane-major packed layout.
enum { kBiasNone = 0, kBiasPlain = 1, kBiasPacked = 2 };

// Biased scores: wherever the weight comes from the table and there is no bias to add.
template <int D, int BC, int BIAS, bool NARROW, int XM>
constexpr bool score_biased() { return XM == kExpTable && !BIAS; }

// How the numerator accumulators are rescaled, and with it the offset they carry: the integer form (ReleaseConst) on 2^30;
// the float form (FloatRelease) on 2^23; or the integer form on 2^23, for what a kernel that uses the float form has to do beyond
// its range.  Moving the offset there and back costs two additions per accumulator and tile (577 tokens with a bias, computed
// weights, tiles of 64: 48.6 us against 54.7), so a kernel that never uses the float form takes the first.
enum { kReleaseInt = 0, kReleaseFloat = 1, kReleaseMoved = 2 };
template <int RELEASE>
constexpr int acc_offset() { return RELEASE == kReleaseInt ? kAccBias : kAccOffset; }

template <bool SB>
__device__ __forceinline__ int smax(int a, int b) { return SB ? (int)max((unsigned)a, (unsigned)b) : max(a, b); }
template <bool SB>
__device__ __forceinline__ int smax3(int a, int b, int c) {
    return SB ? (int)max(max((unsigned)a, (unsigned)b), (unsigned)c) : max(max(a, b), c);
}

//
// LAY selects where the MFMA A operands come from.  kLayPadded: K rows with pitch KROW at sK and V^T
// (columns in result order) with pitch VROW at sV, both written by the staging code of the kernel.
// kLaySwizzled: K and V tiles row-major in LDS exactly as in memory (for 64-byte rows: the four 16-byte
// pieces of row r stored at piece index p ^ ((r >> 2) & 3), which is what keeps both kinds of read
// free of bank conflicts), put there by direct global-to-LDS loads; kx / vx are then this lane's LDS
// byte addresses inside the tile (see swizzled_lane_offsets) and sK, KROW, sV, VROW are unused.
// The V^T operand is read with the transposing 8-bit LDS read of gfx950.
enum { kLayPadded = 0, kLaySwizzled = 1 };

typedef int v2i_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_void;
typedef const __attribute__((address_space(1))) void* glb_void;

// One direct load: the 64 lanes fetch 16 bytes each from g + lane_off (their own offset from a
// uniform address) and the 1 KiB lands at lds_addr + 16 * lane (lds_addr uniform).
// (Spelled out as instructions: for loads it knows to write LDS, the compiler makes the next LDS
// access of the wavefront wait for all of them, while the kernels count them themselves.
// M0 holds the LDS address of such a load; one idle cycle separates writing it from using it.)
__device__ __forceinline__ void load_1k_to_lds(const int8_t* g /* uniform */, int lane_off, int lds_addr /* uniform */) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(lane_off), "s"((glb_void)g) : "memory", "m0");
}

typedef __attribute__((address_space(3))) v2i_t lds_v2i;
typedef const __attribute__((address_space(3))) v4i lds_v4i;

// Four of them for consecutive KiB under one setting of M0 (the offset of the instruction counts on both
// sides): a wavefront issues a direct load per 45 ns when it sets M0 anew each time, per 10 ns when not.
__device__ __forceinline__ void load_4k_to_lds(const int8_t* g /* uniform */, int lane_off, int lds_addr /* uniform */) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\t"
                 "global_load_lds_dwordx4 %1, %2 offset:1024\n\tglobal_load_lds_dwordx4 %1, %2 offset:2048\n\t"
                 "global_load_lds_dwordx4 %1, %2 offset:3072"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(lane_off), "s"((glb_void)g) : "memory", "m0");
}

// ds_read_b64_tr_b8 works on blocks of 16 lanes: lane i of a block receives, as byte j, byte i % 8 of
// the 8 bytes that lane 2 j + i / 8 of the block points to.  With even lanes pointing at features
// f0..f0+7 and odd lanes at f0+8..f0+15 of key row kappa(j), lane i ends up with feature f0 + i of
// the eight keys kappa(0..7): a 16 x 8 piece of V^T.  Two such reads (keys 16 apart) are the 16
// bytes of the A operand of O^T += V^T P^T, with kappa chosen as the row order of the score block
// (k-slot 16 g + 4 a + b  <->  key 8 a + 4 g + b).
// (32 features: 32-byte rows of two pieces, piece p of row r stored at p ^ ((r >> 2) & 1).)
struct SwizzledLane {
    int k_off;   // K / Q operand: row li, 16-byte piece g (k-step 0; k-step 1 is this ^ 32)
    int v_off;   // V^T operand: first transposing read of feature block 0 (block 1 is this ^ 32; keys +16: + 16 rows)
};
template <int D>
__device__ __forceinline__ SwizzledLane swizzled_lane_offsets(int lane) {
    constexpr int M = D / 16 - 1;
    const int li = lane & 31, g = lane >> 5;
    SwizzledLane o;
    o.k_off = li * D + ((g ^ ((li >> 2) & M)) << 4);
    const int li_hi = (lane >> 4) & 1, s = lane & 15, odd = s & 1, j = s >> 1, a = j >> 2, b = j & 3;
    o.v_off = (8 * a + 4 * g + b) * D + ((li_hi ^ ((2 * a + g) & M)) << 4) + 8 * odd;
    return o;
}

// NG: 0, or the number of groups of 8 keys the (ragged) tile has, known at compile time: the tests
// "does this group exist" then cost nothing; n_valid_rt still tells which keys of the last group exist.  NG < 0: at
// most -NG groups and more than -NG / 2 of them; what is in LDS for keys beyond the sequence is then the last key again
// (the maximum stays what it is), and their weights are masked.
template <int D, int BC, int BIAS, int XM, bool SB, bool FULL, bool FIRST, int LAY = kLayPadded, int NG = 0, bool QMAX = false, int RELEASE = kReleaseInt, int MIXED = 0,
          class BeforeV = NothingBeforeV, bool MUL24 = false>
__device__ __forceinline__ void process_tile(RowState<D>& st, const v4i* qreg, const int8_t* sK, int KROW,
                                            const int8_t* sV, int VROW, int n_valid_rt, int x_p,
                                            const int32_t* bias_row /* + c0 */,
                                            const v4i* bpre /* packed bias of this tile already in registers, or null */,
                                            const ExpConst<MUL24>& c, int a_mul, int li, int g,
                                            int kx = 0, int vx = 0, BeforeV before_v = BeforeV()) {
    const v16i zb = offset_block<acc_offset<RELEASE>()>();
    static_assert(!QMAX || RELEASE == kReleaseInt, "its shifts take the offset 2^30");
    constexpr int KSTEPS = D / 32, TB = D / 32, KB = BC / 32;
    constexpr bool KZ = XM == kExpShift0;
    static_assert(!SB || (XM == kExpTable && !BIAS), "biased scores: table mode without bias only");
    static_assert(KB >= 2 && KB <= 4, "one built-in constant per 32-key block");
    // FULL: the tile has all BC kv rows, every "is this group inside the sequence" test below is
    // true at compile time and the tile is one straight line of code.
    constexpr int NGA = NG < 0 ? -NG : NG;
    static_assert(NGA <= BC / 8 && !(FULL && NG != 0), "groups of a ragged tile");
    const int n_valid = FULL ? BC : n_valid_rt;
    // does the 32-key block kb / the group a4 of it exist; does that group reach beyond the sequence
    auto blk_on = [&](int kb) { return NG ? 4 * kb < NGA : 32 * kb < n_valid; };
    auto grp_on = [&](int kb, int a4) { return NG ? 4 * kb + a4 < NGA : 32 * kb + 8 * a4 < n_valid; };
    auto grp_cut = [&](int kb, int a4) {
        return NG > 0 ? 4 * kb + a4 == NG - 1 : NG == 0 && 32 * kb + 8 * a4 + 8 > n_valid;
    };
    // MIXED (look-up mode, 32 features): so many groups of four scores in eight are computed instead of looked up.  A
    // look-up of 64 random bytes costs the LDS of the compute unit 2.1 cycles where they fall into few words, 7.5 where
    // they are spread over a large table (measured: 2.1 and 7.5), its arithmetic nine vector instructions.  At 32
    // features a tile has half the vector work per look-up and the LDS is what runs out first.  us with none, one,
    // two and three groups computed, 96 pairs of 1200 tokens, inputs N(0, sigma^2): sigma 1.0 (table of 12 KB) 36.4 34.2
    // 32.5 32.9, 1.2 (8.5 KB) 32.0 30.6 29.9 31.9, 1.35 (6.7 KB) 28.2 27.9 28.6 31.4, 1.6 (4.8 KB) 24.5 25.8 28.0 31.2: see
    // kRingMixedBytes.  Where a compute unit has one workgroup one group is best, the arithmetic being a longer chain: none, one and
    // two 12.2 12.0 12.3 (32 pairs of 768, tiles of 64), 10.9 10.65 10.75 (of 128); with two workgroups two are (32 of 1600, tiles of
    // 64: 33.5 31.0 30.1).
    // At 64 features computing only costs (40.5 -> 45 us, N = 577).
    static_assert(!MIXED || (XM == kExpTable && D == 32 && LAY == kLaySwizzled), "computed weights beside look-ups");
    constexpr bool MIX = MIXED != 0 && FULL;                    // (a ragged tile would spill)
    auto computed = [&](int kb, int a4) { return MIX && a4 == 3 && (MIXED == 2 || (kb & 1)); };
    // ---- step 1: S^T blocks (32 kv rows x 32 queries each)
    v16i s[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        if (blk_on(kb)) {
            const v4i ka0 = LAY == kLaySwizzled ? *(lds_v4i*)(size_t)(kx + 32 * D * kb)
                                                : *(const v4i*)(sK + (32 * kb + li) * KROW + 16 * g);
            const v16i zs = kb == 0 ? score_offset_block<0>() : kb == 1 ? score_offset_block<1>()
                          : kb == 2 ? score_offset_block<2>() : score_offset_block<3>();
            s[kb] = SB ? __builtin_amdgcn_mfma_i32_32x32x32_i8(ka0, qreg[0], zs, 0, 0, 0)
                       : __builtin_amdgcn_mfma_i32_32x32x32_i8(ka0, qreg[0], v16i{0}, 0, 0, 0);
#pragma unroll
            for (int ks = 1; ks < KSTEPS; ++ks) {
                const v4i ka = LAY == kLaySwizzled ? *(lds_v4i*)(size_t)((kx ^ (32 * ks)) + 32 * D * kb)
                                                   : *(const v4i*)(sK + (32 * kb + li) * KROW + 32 * ks + 16 * g);
                s[kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ka, qreg[ks], s[kb], 0, 0, 0);
            }
        }
    }
    // ---- bias, exclusion and the ragged end of the sequence.  Groups of 4 scores (one result
    //      dword of P) that lie wholly beyond the sequence are skipped everywhere below: the test
    //      32*kb + 8*a4 < n_valid is uniform over the wavefront.
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
            const int cb = 32 * kb + 8 * a4;            // first kv row of the group for g = 0
            if (BIAS == kBiasPacked) {
                // Packed bias: the four values of this lane's group are one 16-byte word, the 64
                // lanes of the wavefront read 1 KiB in a row; columns beyond the sequence hold the
                // exclusion mark already.
                if (grp_on(kb, a4)) {
                    const v4i bv = bpre ? bpre[4 * kb + a4] : *(const v4i*)(bias_row + (4 * kb + a4) * 256);
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        s[kb][4 * a4 + b] = __builtin_elementwise_add_sat(s[kb][4 * a4 + b], bv[b]);
                }
            } else if (BIAS == kBiasPlain && grp_on(kb, a4) && (FULL || !grp_cut(kb, a4))) {
                // plain bias, a group inside the sequence: one load of four dwords (rows need not start on 16
                // bytes; such a load asks for dword alignment only) instead of four loads.  (Column first: the sum of the row
                // and 4 g is otherwise held beside the row, and with 64 features and tiles of 128 up to 60 registers spill: 768 pairs
                // of 197 tokens 43.0 us instead of 36.4.)
                const v4i_a4 bv = *(const v4i_a4*)(bias_row + (cb + 4 * g));
#pragma unroll
                for (int b = 0; b < 4; ++b) s[kb][4 * a4 + b] = __builtin_elementwise_add_sat(s[kb][4 * a4 + b], bv[b]);
            } else if (grp_on(kb, a4) && (BIAS || grp_cut(kb, a4))) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int col = cb + 4 * g + b;
                    const bool beyond = !FULL && col >= n_valid;
                    int val = s[kb][4 * a4 + b];
                    if (BIAS) {
                        // One saturating add does it all: the exclusion mark INT32_MIN drags the
                        // score to the bottom of the range, below every clamp point, so it drops
                        // out of the maximum and gets weight 0 without a compare and select.
                        // (A builtin, not inline assembly: the compiler must see this read of an MFMA
                        // result to insert the wait states the matrix pipeline needs.)
                        const int bv = beyond ? INT32_MIN : bias_row[col];
                        val = __builtin_elementwise_add_sat(val, bv);
                    } else if (beyond) {
                        // below every real score in either representation
                        val = SB ? kMaskedBiased + score_offset_delta(kb) : kNegBig;
                    }
                    s[kb][4 * a4 + b] = val;
                }
            }
        }
    // ---- steps 2,3: row maximum over the tile, running maximum
    // (three-operand maxima, one chain per score block so that they can overlap)
    int m_new = st.m;
    {
        constexpr int BASE = SB ? 1 : 0;             // a block at the common offset
        int mk[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            mk[kb] = kb == BASE ? st.m : (SB ? kMaskedBiased + score_offset_delta(kb) : INT32_MIN);
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4)
                if (grp_on(kb, a4)) {
                    mk[kb] = smax3<SB>(mk[kb], s[kb][4 * a4], s[kb][4 * a4 + 1]);
                    mk[kb] = smax3<SB>(mk[kb], s[kb][4 * a4 + 2], s[kb][4 * a4 + 3]);
                }
        }
        m_new = mk[BASE];
#pragma unroll
        for (int kb = SB ? 0 : 1; kb < KB; ++kb) {       // (from 0 in all variants, a hundred registers were spilled)
            if (kb == BASE) continue;
            if (SB) {
                // (a block that does not exist has no maximum to bring to the common offset)
                if (blk_on(kb)) m_new = smax<SB>(m_new, (int)((unsigned)mk[kb] - (unsigned)score_offset_delta(kb)));
            } else {
                m_new = smax<SB>(m_new, mk[kb]);
            }
        }
    }
    {
        const HalfPair hp = both_halves(m_new);
        m_new = smax<SB>(hp.x, hp.y);
    }
    // ---- QMAX (not Algorithm 1): the reference moves up by whole octaves only.  st.m is the old
    //      reference (a multiple of s_inv, x_shift = 0) and m_new so far the larger of it and the
    //      tile's maximum; n = ceil((m_new - st.m) / s_inv) octaves are added.  The quotient by
    //      multiply-high with ceil(2^30 / s_inv) overshoots by at most one (numerator < 2^24),
    //      which one comparison corrects.
    int n_oct = 0;
    if (QMAX) {
        const unsigned x = ((unsigned)m_new - (unsigned)st.m) + (unsigned)(c.s_inv - 1);
        unsigned q = __umulhi(x << 2, (unsigned)a_mul);
        if (q * (unsigned)c.s_inv > x) q -= 1;
        n_oct = (int)q;
        m_new = st.m + n_oct * c.s_inv;
    }
    const int lo = m_new + c.x_floor;
    const int ml = m_new - c.lead;
    // ---- step 4: max-offset factor alpha, brought to 16 fractional bits
    unsigned alpha16 = 0;
    if (!FIRST && !QMAX) {
        const int a_hat = shift_exp2<KZ, XM != kExpTable>(smax<SB>(st.m, lo), m_new, ml, c);   // (registers are short there)
        alpha16 = min(((unsigned)a_hat * (unsigned)a_mul) >> 14, 65536u);
    }
    // ---- steps 9,10 (the part that concerns the past): ScaleRelease of denominator and numerator.
    //      QMAX: alpha = 2^-n, an arithmetic shift; on the offset representation
    //      floor(x / 2^n) + 2^30 = ((x + 2^30) >> n) + (2^30 - (2^30 >> n)) for n <= 30, and n = 30
    //      stands for every larger n (|x| < 2^26).
    auto release_past = [&]() {
        if (QMAX) {
            const int n = min(n_oct, 30);
            const unsigned addc = (unsigned)kAccBias - ((unsigned)kAccBias >> n);
            st.l = st.l >> n;
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) st.acc[t][v] = (int)(((unsigned)st.acc[t][v] >> n) + addc);
        } else if (RELEASE != kReleaseFloat) {
            constexpr int kMove = kAccBias - acc_offset<RELEASE>();
            const ReleaseConst ri = make_release(alpha16);
            st.l = release_l(st.l, ri);
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) st.acc[t][v] = release_acc(st.acc[t][v] + kMove, ri) - kMove;
        } else {
            const FloatRelease rf = make_float_release(alpha16);
            st.l = release_l(st.l, rf);
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) st.acc[t][v] = release_acc(st.acc[t][v], rf);
        }
    };
    v4i pk[KB];
    int rowsum = 0;
    if (XM == kExpTable) {
        // ---- steps 5,6 by table: issue every look-up of the tile, rescale the accumulators while
        //      the LDS answers, then pack.  Index 0 of the table is the weight 0 of everything at
        //      or below -x_p (excluded scores included).
        const unsigned x_p_v = (unsigned)to_vgpr(x_p);
        const unsigned edge = (unsigned)m_new - x_p_v;       // score_biased: m + 2^30 - x_p > 0
        const float addend0 = index_addend(edge), scale0 = __int_as_float(to_vgpr((int)kIndexScale));
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const unsigned edge_kb = edge + (unsigned)score_offset_delta(kb);   // (the block's own offset)
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4)
                if (grp_on(kb, a4)) {
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        // Saturating subtractions are fast-class instructions; as builtins, because
                        // they read MFMA results.
                        const unsigned sv = (unsigned)s[kb][4 * a4 + b];
                        const unsigned idx = SB && kb == 0 && (FULL || NG) ? float_index((int)sv, scale0, addend0)
                                           : SB ? __builtin_elementwise_sub_sat(sv, edge_kb)
                                                : __builtin_elementwise_sub_sat(x_p_v, (unsigned)m_new - sv);
                        s[kb][4 * a4 + b] = computed(kb, a4) ? (int)idx : table_weight(idx);
                    }
                }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (MIX) {
            const unsigned neg_xpk = (unsigned)to_vgpr(-(x_p << c.k));
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int a4 = 0; a4 < 4; ++a4)
                    if (computed(kb, a4) && grp_on(kb, a4)) {
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const int xs = (int)(((unsigned)s[kb][4 * a4 + b] << c.k) + neg_xpk);
                            s[kb][4 * a4 + b] = (int)c.weight(shift_exp2_shifted(xs, xs + c.lead_v, c));
                        }
                    }
        }
        if (!FIRST) release_past();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            pk[kb] = v4i{0, 0, 0, 0};
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4)
                if (grp_on(kb, a4)) {
                    const unsigned p0 = (unsigned)s[kb][4 * a4], p1 = (unsigned)s[kb][4 * a4 + 1];
                    const unsigned p2 = (unsigned)s[kb][4 * a4 + 2], p3 = (unsigned)s[kb][4 * a4 + 3];
                    unsigned w = computed(kb, a4) ? pack_byte3(p0, p1, p2, p3)
                                                : FULL || NG ? pack_weights(p0, p1, p2, p3) : pack_byte<0>(p0, p1, p2, p3);
                    if (NG < 0 && 4 * kb + a4 >= NGA / 2) w &= first_bytes(n_valid - (32 * kb + 8 * a4 + 4 * g));
                    pk[kb][a4] = (int)w;
                    rowsum = add_bytes(w, rowsum);   // step 7
                }
        }
        {
            const HalfPair hp = both_halves(rowsum);
            rowsum = hp.x + hp.y;
        }
        st.l += rowsum;                                                                    // step 9
    } else {
        // ---- steps 5,6,7: score intensity, requantisation to int8 (Eq. 10), row sum
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            pk[kb] = v4i{0, 0, 0, 0};
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4)
                if (grp_on(kb, a4)) {
                    unsigned pr[4];
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const int y = shift_exp2<KZ>(max(s[kb][4 * a4 + b], lo), m_new, ml, c);
                        pr[b] = c.weight(y);
                    }
                    const unsigned w = pack_byte3(pr[0], pr[1], pr[2], pr[3]);
                    pk[kb][a4] = (int)w;
                    rowsum = add_bytes(w, rowsum);
                }
        }
        {
            const HalfPair hp = both_halves(rowsum);
            rowsum = hp.x + hp.y;
        }
        // Keep the phases apart: letting the scheduler overlap the rescale below with the
        // element-wise work above only lengthens live ranges (spills) without gaining issue slots.
        __builtin_amdgcn_sched_barrier(0);
        // ---- steps 9,10: ScaleRelease of the running denominator and numerator
        if (FIRST) {
            st.l = rowsum;
        } else {
            release_past();
            st.l += rowsum;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    before_v();
    // ---- step 8: O^T += V_j^T P^T (the first tile starts the accumulators at their offset)
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
            if (blk_on(kb)) {
                v4i va;
                if (LAY == kLaySwizzled) {
                    const int va_addr = (vx ^ (32 * t)) + 32 * D * kb;
                    const v2i_t lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(size_t)va_addr);
                    const v2i_t hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(size_t)(va_addr + 16 * D));
                    va = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
                } else {
                    va = *(const v4i*)(sV + (32 * t + li) * VROW + 32 * kb + 16 * g);
                }
                st.acc[t] = (FIRST && kb == 0) ? __builtin_amdgcn_mfma_i32_32x32x32_i8(va, pk[kb], zb, 0, 0, 0)
                                               : __builtin_amdgcn_mfma_i32_32x32x32_i8(va, pk[kb], st.acc[t], 0, 0, 0);
            }
    st.m = m_new;
}

// Step 11: integer normalisation floor(O / l) (or nearest), saturated to int8, without a division
// per element.  With u = O + 128 l clamped to [0, 256 l), t = floor(u / l) lies in [0, 255] and
// floor(O / l) saturated to [-128, 127] equals t - 128, i.e. byte t ^ 0x80.  l is normalised to
// l' = l << z in (2^(L-1), 2^L] and R = ceil(2^(2L+8) / l'); then floor(u' R / 2^(2L+8)) is exact
// for every u' < 256 l' because u' (R l' - 2^(2L+8)) < 2^(L+8) 2^L.  L = 16 or 20 puts the quotient
// into byte 1 or 2 of the high product word.  Nearest: floor((2 O + l) / (2 l)), same scheme with
// numerator 2 O + l and denominator 2 l.
// min(max(u, 0), hi) for hi >= 0 as one instruction (the median of three).  u is the result of an
// ordinary vector instruction, not of a matrix instruction, and the output is tied to it (the rules
// for inline assembly next to to_vgpr).
__device__ __forceinline__ int clamp_0(int u, int hi) {
    int r = u;
    asm("v_med3_i32 %0, %0, 0, %1" : "+v"(r) : "v"(hi));
    return r;
}

// normalise_words leaves the lane's contiguous half of the output row (D / 2 bytes: lane g = 0 the
// first half, g = 1 the second) in out[0 .. D/32); normalise_store also writes it.
// OFFSET: the offset the accumulators carry.
template <int D, int L, int OFFSET>
__device__ __forceinline__ void normalise_words(const RowState<D>& st, bool round_nearest, v4i* out) {
    constexpr int TB = D / 32;
    static_assert(L == 16 || L == 20, "quotient must be byte aligned");
    const int rs = round_nearest ? 1 : 0;
    const bool empty = st.l == 0;
    const unsigned dsafe = empty ? 1u : ((unsigned)st.l << rs);
    const int z = L - (32 - __clz((int)(dsafe - 1)));          // dsafe << z in (2^(L-1), 2^L]
    const unsigned dn = dsafe << z;
    const unsigned R = recip_ceil<L>(dn);
    const int u_max = (int)(256u * dn) - 1;
    const int zz = z + rs;
    // The accumulators carry their offset (ReleaseConst); it is taken out, modulo 2^32, together
    // with the addition of 128 l.
    int bias_z = (int)(((128u * dsafe + (round_nearest ? (unsigned)st.l : 0u)) << z) - ((unsigned)OFFSET << zz));
    asm volatile("" : "+v"(bias_z));     // (kept as one addend: otherwise the offset is subtracted from every element first)
    // word[j]: features 8 j + 4 g + (0..3) of this lane's row, j = 4 t + a4
    unsigned word[4 * TB];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
            unsigned hi[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                int u = (st.acc[t][4 * a4 + b] << zz) + bias_z;
                u = clamp_0(u, u_max);
                hi[b] = __umulhi((unsigned)u, R);
            }
            const unsigned w = pack_byte<(2 * L + 8 - 32) / 8>(hi[0], hi[1], hi[2], hi[3]) ^ 0x80808080u;
            word[4 * t + a4] = empty ? 0u : w;
        }
    // The two lanes of a row hold alternate dwords of it.  Swapping the second half of the row of
    // lane g = 0 against the first half of lane g = 1 (one cross-lane swap per dword) leaves each
    // lane with one contiguous half of the row, written with 16-byte stores: dword-sized stores
    // scattered over 32 rows per instruction cost more time than the whole computation.
    constexpr int HALF = 2 * TB;   // dwords a lane owns after the swap (as many as before it)
    unsigned ev[HALF], od[HALF];   // even / odd dwords of this lane's half
#pragma unroll
    for (int j = 0; j < HALF; ++j) {
        const auto sw = __builtin_amdgcn_permlane32_swap(word[j], word[HALF + j], false, false);
        ev[j] = sw[0];
        od[j] = sw[1];
    }
#pragma unroll
    for (int q = 0; q < HALF / 2; ++q)
        out[q] = v4i{(int)ev[2 * q], (int)od[2 * q], (int)ev[2 * q + 1], (int)od[2 * q + 1]};
}

// The same (rounding down, denominators up to kFloatNormaliseMaxL) with floats, see FloatQuotient: three instructions per element,
// two of which issue beside integer ones, instead of nearly four, and no Newton iteration: 768 pairs of 197 tokens 16.1 -> 15.6 us,
// 256 of 577 20.4 -> 19.7, windows (12288 pairs of 49) 19.2 -> 17.9.  v_cvt_pk_u8_f32 floors, saturates to [0, 255] and packs.
template <int D, int OFFSET>
__device__ __forceinline__ void float_normalise_words(const RowState<D>& st, v4i* out) {
    constexpr int TB = D / 32, HALF = 2 * TB;
    const FloatQuotient<OFFSET> quotient(st.l == 0 ? 0.0f : __builtin_amdgcn_rcpf((float)st.l));
    const float scale = __int_as_float(to_vgpr((int)FloatQuotient<OFFSET>::kScale));
    unsigned word[4 * TB];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
            unsigned w = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) w = __builtin_amdgcn_cvt_pk_u8_f32(quotient(st.acc[t][4 * a4 + b], scale), b, w);
            word[4 * t + a4] = w ^ 0x80808080u;
        }
#pragma unroll
    for (int q = 0; q < HALF / 2; ++q) {
        unsigned ev[2], od[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const auto sw = __builtin_amdgcn_permlane32_swap(word[2 * q + k], word[HALF + 2 * q + k], false, false);
            ev[k] = sw[0];
            od[k] = sw[1];
        }
        out[q] = v4i{(int)ev[0], (int)od[0], (int)ev[1], (int)od[1]};
    }
}

// The same for n quads of four features of one row (accumulators with their offset).
template <int L, int NQ>
__device__ __forceinline__ void normalise_quads(const v4i* acc, int l, bool round_nearest, unsigned* out) {
    const int rs = round_nearest ? 1 : 0;
    const bool empty = l == 0;
    const unsigned dsafe = empty ? 1u : ((unsigned)l << rs);
    const int z = L - (32 - __clz((int)(dsafe - 1)));
    const unsigned dn = dsafe << z;
    const unsigned R = recip_ceil<L>(dn);
    const int u_max = (int)(256u * dn) - 1, zz = z + rs;
    const int bias_z = (int)(((128u * dsafe + (round_nearest ? (unsigned)l : 0u)) << z) - ((unsigned)kAccBias << zz));
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        unsigned hi[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) hi[b] = __umulhi((unsigned)clamp_0((acc[q][b] << zz) + bias_z, u_max), R);
        const unsigned w = pack_byte<(2 * L + 8 - 32) / 8>(hi[0], hi[1], hi[2], hi[3]) ^ 0x80808080u;
        out[q] = empty ? 0u : w;
    }
}

template <int D, int L, int OFFSET>
__device__ __forceinline__ void normalise_store(const RowState<D>& st, int8_t* Orow, int g, bool round_nearest) {
    v4i w[D / 32];
    if (OFFSET == kAccOffset && !round_nearest && (L == 16 || __builtin_amdgcn_ballot_w64(st.l > kFloatNormaliseMaxL) == 0))
        float_normalise_words<D, OFFSET == kAccOffset ? OFFSET : kAccOffset>(st, w);
    else
        normalise_words<D, L, OFFSET>(st, round_nearest, w);
    int8_t* dst = Orow + g * (D / 2);
#pragma unroll
    for (int q = 0; q < D / 32; ++q) *(v4i*)(dst + 16 * q) = w[q];
}


// Constants of the head that (batch, head) pair bh belongs to.  bh is uniform over the wavefront,
// so these are scalar loads from the kernel arguments.
// With dynamic quantisation they were computed on the GPU and live in device memory: read field
// by field into scalar registers (selecting between the two structures by pointer would turn every
// access, the table loads included, into generic-address loads).
__device__ __forceinline__ QflashHeadConsts head_consts_or_dev(const QflashLaunchArgs& a, QflashHeadConsts h) {
    if (a.hc_dev) {
        const int* g = (const int*)a.hc_dev;     // x_shift, s_inv, exp_mul, p_mul, p_shift, a_mul, x_floor
        h.x_shift = __builtin_amdgcn_readfirstlane(g[0]);
        h.s_inv = __builtin_amdgcn_readfirstlane(g[1]);
        h.exp_mul = __builtin_amdgcn_readfirstlane(g[2]);
        h.p_mul = __builtin_amdgcn_readfirstlane(g[3]);
        h.p_shift = __builtin_amdgcn_readfirstlane(g[4]);
        h.a_mul = __builtin_amdgcn_readfirstlane(g[5]);
        h.x_floor = __builtin_amdgcn_readfirstlane(g[6]);
        // the table, if the GPU built one for these constants (lut_bytes == 0: none)
        h.lut_xp = __builtin_amdgcn_readfirstlane(g[7]);
        h.lut_bytes = __builtin_amdgcn_readfirstlane(g[8]);
        if (h.lut_bytes > a.lut_bytes_max) h.lut_bytes = 0;      // (the launch has no room for it)
        const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane(g[10]), hi = (unsigned)__builtin_amdgcn_readfirstlane(g[11]);
        h.lut = (const uint8_t*)(((unsigned long long)hi << 32) | lo);
    }
    return h;
}
__device__ __forceinline__ QflashHeadConsts head_consts(const QflashLaunchArgs& a, int) {
    return head_consts_or_dev(a, qflash_unpack_head(a.one, a.lut_base));
}
// (An index, and no choice between hw[] and `one`: that puts a branch into the path of launches with one set of constants, 1104 pairs of
// 197 tokens 27.9 us against 27.7, windows of 144 with a plain bias, 768 pairs 8.94 against 8.84, 6144 38.7 against 38.5.)
__device__ __forceinline__ QflashHeadConsts head_consts(const QflashKernelArgs& a, int bh) {
    return head_consts_or_dev(a, qflash_unpack_head(a.hw[a.per_head ? bh % a.H : 0], a.lut_base));
}
// Of head h of a launch with per-head constants.
__device__ __forceinline__ QflashHeadConsts own_head_consts(const QflashKernelArgs& a, int h) {
    return qflash_unpack_head(a.hw[h], a.lut_base);
}
static_assert(offsetof(QflashHeadConsts, x_floor) == 24 && offsetof(QflashHeadConsts, lut_xp) == 28 &&
              offsetof(QflashHeadConsts, lut_bytes) == 32 && offsetof(QflashHeadConsts, lut) == 40,
              "field order read by head_consts");

// Where this lane's bias values start.  Plain layout [bias_B,bias_H,N,N]: the lane's row (lanes
// beyond the sequence read row 0; their results are never stored).  Packed layout
// [bias_B*bias_H][ceil(N/32) row blocks][ceil(N/32) column blocks][4 groups][64 lanes][4]: the
// 16-byte word of lane (li, g) in group a4 of column block cb holds
// bias[32*rb + li][32*cb + 8*a4 + 4*g + 0..3], which is exactly what the lane adds to its four
// scores of that group, so one instruction of the wavefront reads 1 KiB in a row.
__device__ __forceinline__ const int32_t* bias_lane_base(const QflashLaunchArgs& a, int bh, int row0, int i,
                                                        int li, int g) {
    const int b = bh / a.H, h = bh % a.H, N = a.N;
    const unsigned slice32 = (unsigned)(b % a.bias_B) * (unsigned)a.bias_H + (unsigned)(h % a.bias_H);   // (below 2^31)
    asm volatile("" :: "s"(slice32));                     // (made here, ahead of a change of the rounding mode: round_down)
    const size_t slice = slice32;
    if (a.bias_packed) {
        const int nb = (N + 31) / 32;
        return a.bias + ((slice * nb + (size_t)min(row0 / 32, nb - 1)) * nb) * 1024 + 4 * (32 * g + li);
    }
    return a.bias + slice * N * N + (size_t)(i < N ? i : 0) * N;
}

}  // namespace
