// Scales, integer constants and weight table of a call with dynamic quantisation, made on the GPU: shared by the
// quantising kernel and the attention kernel that quantises on the way in.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qflash.h"
#include "qflash_internal.h"
#include "qflash_derive.h"
#include "qflash_device.h"

namespace {

// Scales and constants from the three maxima (one thread).  *unit: real value of one integer score unit.
__device__ void derive_on_device(const float am[3], double sqrt_d, int out_round, QflashHeadConsts* hc,
                                 qflash_dynamic_info* info, double* unit) {
    double s[3];
    for (int t = 0; t < 3; ++t) s[t] = am[t] == 0.0f ? 1.0 : (double)am[t] / 127.0;   // all-zero tensor: scale 1
    if (unit) *unit = __ddiv_rn(__dmul_rn(s[0], s[1]), sqrt_d);
    qflash_params p;
    int status = qflash_derive_params(s[0], s[1], sqrt_d, &p);
    if (status == QFLASH_OK) {
        p.out_round = out_round;
        if (!qflash_fill_head_consts(p, hc)) status = QFLASH_ERR_PARAM;
    }
    if (status != QFLASH_OK) {
        // Scales outside the supported window: the attention kernel runs on safe constants (those
        // of a mid-range scale) with the requantisation multiplier set to 0, so that every weight is
        // 0, every denominator is 0 and the output is all zeros (Algorithm 1 with l = 0); the status
        // says why.
        (void)qflash_derive_params(0.03, 0.03, sqrt_d, &p);
        p.out_round = out_round;
        (void)qflash_fill_head_consts(p, hc);
        hc->p_mul = 0;
    }
    if (info) {
        info->sQ = s[0]; info->sK = s[1]; info->sV = s[2];
        info->params = p;
        info->status = status;
    }
}

// Records in *hc a weight table of x_p + 1 entries (the host's rule), padded to 16, if that is at most table_max bytes.
__device__ __forceinline__ void reserve_table(QflashHeadConsts* hc, const uint8_t* table, int table_max) {
    const long long x_p = qflash_table_span(hc->s_inv, hc->x_shift, max(hc->p_mul, 1), hc->p_shift);
    const long long n_padded = (x_p + 1 + 15) & ~15ll;
    const bool fits = n_padded <= (long long)table_max;
    hc->lut = fits ? table : nullptr;
    hc->lut_bytes = fits ? (int)n_padded : 0;
    hc->lut_xp = fits ? (int)x_p : 0;
}

// A bias in real units ---------------------------------------------------------------------------

// A bias value in the score unit: clip(floor(x / unit + 0.5)), in float64 with one rounding per operation.  The product
// with the reciprocal decides unless it is within 2^-24 of the edge (its error is below 2^-29 where the
// clip does not decide), which spares a division of 30 instructions.
__device__ __forceinline__ int bias_word(float x, double unit, double inv) {
    double t = __dadd_rn(__dmul_rn((double)x, inv), 0.5);
    double f = floor(t);
    const double frac = t - f;
    if (!(frac > 0x1p-24 && frac < 1.0 - 0x1p-24)) {
        t = __dadd_rn(__ddiv_rn((double)x, unit), 0.5);
        f = floor(t);
    }
    return (int)fmin(fmax(f, -1048575.0), 1048575.0);
}

// For the attention kernels that quantise on the way in ------------------------------------------

// The partial maxima of the three tensors (at most 256 each), one to four per lane: loaded first, reduced when they
// are needed.  Every wavefront does this for itself.
struct PartialMaxima {
    float part[3][4];
    __device__ __forceinline__ void load(const QflashLaunchArgs& a) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int k = 0; k < 4; ++k) part[t][k] = a.dyn_partial[t * a.dyn_partials + min(lane + 64 * k, a.dyn_partials - 1)];
    }
    __device__ __forceinline__ float maximum(int t) const {
        float m = fmaxf(fmaxf(part[t][0], part[t][1]), fmaxf(part[t][2], part[t][3]));
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
        return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(m)));
    }
    __device__ __forceinline__ float factor(int t) const {
        const float am = maximum(t);
        return am == 0.0f ? 0.0f : __fdiv_rn(127.0f, am);
    }
};

typedef float v4f __attribute__((ext_vector_type(4)));

// Four elements to four bytes: clip, then round half to even by adding 1.5 * 2^23 (the low byte of the sum
// is the integer; the clip, between the two roundings, also keeps them from becoming one).
__device__ __forceinline__ int quantise4(v4f x, float r) {
    unsigned q[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float c = __builtin_amdgcn_fmed3f(__fmul_rn(x[e], r), -127.0f, 127.0f);
        q[e] = __float_as_uint(__fadd_rn(c, 12582912.0f));
    }
    return (int)(__builtin_amdgcn_perm(q[1], q[0], 0x0c0c0400u) | __builtin_amdgcn_perm(q[3], q[2], 0x04000c0cu));
}

// One lane: constants and score unit from the maxima, to LDS at hc_base (kDynConstBytes).
typedef __attribute__((address_space(3))) int dyn_lds_int;
__device__ __forceinline__ void derive_to_lds(const QflashLaunchArgs& a, const float (&am)[3], int hc_base) {
    QflashHeadConsts h;
    double unit;
    derive_on_device(am, a.dyn_sqrt_d, a.out_round, &h, blockIdx.x == 0 ? a.dyn_info : nullptr, &unit);
    reserve_table(&h, nullptr, a.lut_bytes_max);
    const long long u = __double_as_longlong(unit);
    const int w[11] = {h.x_shift, h.s_inv, h.exp_mul, h.p_mul, h.p_shift, h.a_mul, h.x_floor, h.lut_xp, h.lut_bytes, (int)u, (int)(u >> 32)};
#pragma unroll
    for (int k = 0; k < 11; ++k) *(dyn_lds_int*)(size_t)(hc_base + 4 * k) = w[k];
}
__device__ __forceinline__ QflashHeadConsts consts_from_lds(int hc_base) {
    int w[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) w[k] = __builtin_amdgcn_readfirstlane(*(dyn_lds_int*)(size_t)(hc_base + 4 * k));
    QflashHeadConsts hc;
    hc.x_shift = w[0]; hc.s_inv = w[1]; hc.exp_mul = w[2]; hc.p_mul = w[3]; hc.p_shift = w[4]; hc.a_mul = w[5];
    hc.x_floor = w[6]; hc.lut_xp = w[7]; hc.lut_bytes = w[8];
    hc.lut = nullptr;
    return hc;
}
__device__ __forceinline__ double unit_from_lds(int hc_base) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane(*(dyn_lds_int*)(size_t)(hc_base + 36));
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane(*(dyn_lds_int*)(size_t)(hc_base + 40));
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}
// Share `part` of `parts` wavefronts in the weight table of hc, at LDS address lds0.
__device__ __forceinline__ void table_to_lds(const QflashHeadConsts& hc, int lds0, int part, int parts) {
    const ExpConst<> c = make_exp_const(hc);
    for (int i = 4 * (64 * part + (int)(threadIdx.x & 63)); i < hc.lut_bytes; i += 4 * 64 * parts) {
        unsigned w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) w |= (i + e <= hc.lut_xp ? table_entry(i + e, hc.lut_xp, hc, c) : 0u) << (8 * e);
        *(dyn_lds_int*)(size_t)(lds0 + i) = (int)w;
    }
}

}  // namespace
