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

}  // namespace
