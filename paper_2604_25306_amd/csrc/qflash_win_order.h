// The order in which windowed launches take their (batch, head) pairs.  No HIP in it: tests/test_win_order.py compiles this file for the
// host and walks it.
#pragma once
#include "qflash_internal.h"

#if defined(__HIPCC__)
#define QF_ORDER_FN __host__ __device__ __forceinline__
#else
#define QF_ORDER_FN inline
#endif

namespace {

struct WinPair {      // where a run stands: pair t of the launch order
    int s_idx;        // bias slice = wb * bias_H + hb
    int wb, hb;       // batch and head index of the slice inside the bias
    int i, j;         // replica of the slice: batch step, head step
};

// The order of the pairs: those of one bias slice one after the other.
struct WinOrder {
    int H, bias_B, bias_H, Rb, Rh;      // Rb, Rh: replicas of a slice (the host checked divisibility)
    unsigned inv_R, inv_Rh, inv_bH;
    QF_ORDER_FN explicit WinOrder(const QflashLaunchArgs& a, bool has_bias) {
        H = a.H;
        bias_B = has_bias ? a.bias_B : 1;
        bias_H = has_bias ? a.bias_H : 1;
        Rb = a.win_rb;
        Rh = a.win_rh;
        inv_R = a.win_inv_r;
        inv_Rh = a.win_inv_rh;
        inv_bH = a.win_inv_bh;
    }
    QF_ORDER_FN WinPair at(int t) const {
        WinPair p;
        unsigned r, j, hb;
        p.s_idx = (int)qflash_divide((unsigned)t, (unsigned)(Rb * Rh), inv_R, &r);
        p.i = (int)qflash_divide(r, (unsigned)Rh, inv_Rh, &j);
        p.wb = (int)qflash_divide((unsigned)p.s_idx, (unsigned)bias_H, inv_bH, &hb);
        p.j = (int)j;
        p.hb = (int)hb;
        return p;
    }
    QF_ORDER_FN int pair_index(const WinPair& q) const {      // (batch, head) pair number b * H + h
        return (q.wb + q.i * bias_B) * H + q.hb + q.j * bias_H;
    }
    QF_ORDER_FN void advance(WinPair& q) const {              // (divisions only once per run, above)
        if (++q.j == Rh) {
            q.j = 0;
            if (++q.i == Rb) {
                q.i = 0;
                ++q.s_idx;
                if (++q.hb == bias_H) { q.hb = 0; ++q.wb; }
            }
        }
    }
    QF_ORDER_FN int left_in_slice(const WinPair& q) const { return (Rb - q.i) * Rh - q.j; }
};

}  // namespace
