// gfx950 kernel of the integer-only fused attention forward pass (Algorithm 1) for windowed
// attention: sequences of 33 to 64 tokens with 32 features per head (7 x 7 windows), one KV tile, an
// optional additive bias, packed or plain (relative-position bias, shifted-window mask).
//
// Such a layer is thousands of tiny independent problems (6 KB of Q, K, V, O per pair, but 16 KB of
// bias), so what matters is what is NOT done per pair.  The kernel is persistent: one workgroup of up
// to 16 wavefronts per compute unit, the weight table staged into LDS once per workgroup, and every
// wavefront on its own from then on -- no barrier, no flag, no shared K/V:
//   - a wavefront owns one half of the query rows (rows 0-31 or 32-63) of a run of consecutive
//     pairs.  Pairs are numbered so that a run shares one bias slice (same window position and head
//     in consecutive images); the 32 bias words of the lane stay in registers, already offset, and
//     serve as the accumulator input of the first matrix product: adding the bias costs nothing.
//   - K, V and the wavefront's 32 query rows go to private LDS buffers (5 KiB, two sets,
//     alternating) by direct global-to-LDS loads, one pair ahead of their use, row-major as in
//     memory.  K and Q rows are MFMA operands exactly as they lie there (lane (l % 32, l / 32) reads
//     bytes 16 (l / 32) .. +15 of row l % 32); the V^T operand is read with the transposing 8-bit
//     LDS read.  No staging registers, no transposition in the vector ALU, no LDS write
//     instruction, and nothing in flight that the compiler has to count: the only wait of an
//     iteration is the one at its top.
// Keys beyond the sequence and excluded pairs carry a large negative accumulator input
// (-2^29 before the offset), far below every real score, so they fall out of the maximum and get
// weight 0 without a test.  Scores carry the offset 2^30 (see qflash_tile.h), which turns the
// table index into one saturating subtraction.  12288 pairs of 49 tokens, bias packed, a call: 19.2 -> 18.1 us with
// the normalisation and packing on the float units, 17.5 with the first requests early (below); 77 MB, 14.9 at the rate of a copy.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "qflash_counters.h"
#include "qflash_derive_device.h"
#include "qflash_launch.h"
#include "qflash_tile.h"
#include "qflash_win_order.h"

// (M0 is written by the direct loads below and declared as clobbered)
#pragma clang diagnostic ignored "-Winline-asm"

namespace {

extern __shared__ __align__(1024) int8_t smem_win[];

constexpr int kWinSetBytes = 5 * 1024;     // V, K and 32 query rows of one pair
constexpr int kWinExcluded = -(1 << 29);   // stands for "takes no part" in the offset representation

// The attention of one half of a pair's query rows.  q_addr, k_addr, v_addr: LDS addresses of this lane's operand
// rows; cb: accumulator input; operands_read() is called when the last LDS read of the pair has been issued.
template <int XM, class Done>
__device__ __forceinline__ v4i win_half(int q_addr, int k_addr, int v_addr, const v16i (&cb)[2], const QflashHeadConsts& hc,
                                        const ExpConst<>& c, bool out_round, Done operands_read) {
    constexpr int D = 32;
    constexpr bool KZ = XM == kExpShift0;
    // ---- step 1: S^T + bias (two blocks of 32 keys x 32 queries)
    const v4i q_cur = *(lds_v4i*)(size_t)(q_addr);
    v16i s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const v4i k_cur = *(lds_v4i*)(size_t)(k_addr + 1024 * kb);
        s[kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(k_cur, q_cur, cb[kb], 0, 0, 0);
    }
    // ---- steps 2, 3: row maximum (unsigned: every value carries 2^30), never below the initial maximum
    int m_new;
    {
        unsigned mk[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            mk[kb] = kb == 0 ? (unsigned)kMInit + (unsigned)kAccBias : 0u;
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4) {
                mk[kb] = max(max(mk[kb], (unsigned)s[kb][4 * a4]), (unsigned)s[kb][4 * a4 + 1]);
                mk[kb] = max(max(mk[kb], (unsigned)s[kb][4 * a4 + 2]), (unsigned)s[kb][4 * a4 + 3]);
            }
        }
        const HalfPair hp = both_halves((int)max(mk[0], mk[1]));
        m_new = (int)max((unsigned)hp.x, (unsigned)hp.y);
    }
    // ---- steps 5-7: weights, packed four to a dword (the B operand of the second product), row sum
    v4i pk[2];
    int rowsum = 0;
    if (XM == kExpTable) {
        const unsigned edge = (unsigned)m_new - (unsigned)to_vgpr(hc.lut_xp);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                s[kb][v] = table_weight(__builtin_elementwise_sub_sat((unsigned)s[kb][v], edge));
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4) {
                const unsigned w = pack_weights((unsigned)s[kb][4 * a4], (unsigned)s[kb][4 * a4 + 1],
                                                (unsigned)s[kb][4 * a4 + 2], (unsigned)s[kb][4 * a4 + 3]);
                pk[kb][a4] = (int)w;
                rowsum = add_bytes(w, rowsum);
            }
    } else {
        const int lo = m_new + c.x_floor;
        const int ml = m_new - c.lead;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4) {
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
    RowState<D> st;
    {
        const HalfPair hp = both_halves(rowsum);
        st.l = hp.x + hp.y;
    }
    st.m = m_new;
    // ---- step 8: O^T = V^T P^T, the V^T operand read transposed from the row-major V in LDS
    {
        v16i acc = offset_block<kScoreOffset0>();
        v4i va[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const v2i_t lo2 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(size_t)(v_addr + 1024 * kb));
            const v2i_t hi2 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(size_t)(v_addr + 1024 * kb + 512));
            va[kb] = __builtin_shufflevector(lo2, hi2, 0, 1, 2, 3);
        }
        operands_read();
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[kb], pk[kb], acc, 0, 0, 0);
        st.acc[0] = acc;
    }
    // ---- step 11
    v4i o;
    if (!out_round) float_normalise_words<D, kScoreOffset0>(st, &o);
    else normalise_words<D, 16, kScoreOffset0>(st, true, &o);
    return o;
}

// Lane part of the LDS address of the V^T operand (read with the transposing 8-bit read, see qflash_tile.h).
__device__ __forceinline__ int win_v_lane(int lane) {
    const int li_hi = (lane >> 4) & 1, s = lane & 15, odd = s & 1, jj = s >> 1, aa = jj >> 2, bb = jj & 3;
    return (8 * aa + 4 * (lane >> 5) + bb) * 32 + 16 * li_hi + 8 * odd;
}

template <int XM, bool PLAIN>
__device__ __forceinline__ void win_body(const QflashLaunchArgs& a) {
    constexpr int D = 32;
    round_down();
    const int N = a.N;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_waves = (int)(blockDim.x >> 6);
    const int g = lane >> 5, li = lane & 31;
    const QflashHeadConsts hc = head_consts(a, 0);
    const ExpConst<> c = make_exp_const<XM != kExpTable>(hc);

    // ---- LDS: [weight table, a.win_table_lds bytes][wavefront w: two sets of V (2 KiB), K (2 KiB),
    //      Q (1 KiB)]; the dynamic LDS is the only LDS of the kernel, so the table index is its address
    const int lds0 = (int)(size_t)(lds_void)smem_win;
    const int tbytes = XM == kExpTable ? a.win_table_lds : 0;
    if (XM == kExpTable) {
        for (int it = wave; it < ((hc.lut_bytes + 1023) >> 10); it += n_waves)
            load_1k_to_lds((const int8_t*)hc.lut + 1024 * it, 16 * lane, lds0 + 1024 * it);
    }
    // The only barrier: the table is in place.  The first pair's five loads are requested ahead of it, behind those of the table, and stay in
    // flight across it: 384 pairs with a packed bias 3.73 -> 3.36 us, 4608 of 64 tokens 12.5 -> 12.1.  Behind it (late) where a compute
    // unit has more than eight wavefronts and their bias would come behind the K and V of all of them: with a plain bias, as
    // many bytes in scattered pieces, and where every wavefront has one pair only.  By turns as well, with a plain bias: that of the first
    // wavefronts then comes ahead of the K and V of the last.  Inputs from memory: 1632 pairs of 64 tokens, plain, 9.26 us, late 8.97, by
    // turns 8.62; 4608 13.3, 13.3, 12.9; packed, 1632 of 64 7.84, late 7.59, 1536 of 64 equal.  (128 to 450 cycles a turn measured the
    // same.  The bias ahead of the barrier as well: 5472 pairs 10.6 -> 11.3, every wavefront then waits for the last of all loads.)
    const bool late = a.win_streams > 4 && (PLAIN || a.win_chunk == 1);
    auto table_in_place = [late] {
        if (XM != kExpTable) return;
        if (late) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
        __syncthreads();
    };

    // ---- this wavefront's run of pairs
    const int half = wave & 1;
    const int sid = blockIdx.x * a.win_streams + (wave >> 1);
    const int T = a.B * a.H;
    const int t0 = sid * a.win_chunk, t1 = min(t0 + a.win_chunk, T);
    if ((wave >> 1) >= a.win_streams || t0 >= t1) {
        if (XM == kExpTable) {            // (its share of the table, none of the five)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
        return;
    }

    const bool has_bias = a.bias != nullptr;
    const WinOrder order(a, has_bias);
    WinPair p = order.at(t0);
    // ---- per-lane offsets (bytes).  In memory: the two 1 KiB pieces of K and V of a pair and the
    //      1 KiB of this half's query rows, each clamped to the pair's last 16 bytes (what lands in
    //      rows beyond the sequence meets weight 0 or is never stored).  In LDS: operand rows, the
    //      V^T operand.
    const int row = 32 * half + li;
    const int voff0 = min(16 * lane, N * D - 16), voff1 = min(1024 + 16 * lane, N * D - 16);
    const int qoff = min(1024 * half + 16 * lane, N * D - 16);
    const int wbuf = lds0 + tbytes + wave * (2 * kWinSetBytes);
    const int op_lane = 32 * li + 16 * g;
    const int v_lane = win_v_lane(lane);
    const size_t pair_bytes = (size_t)N * D;

    auto issue_loads = [&](const WinPair& q, int parity) {
        const size_t off = (size_t)order.pair_index(q) * pair_bytes;
        const int set = wbuf + kWinSetBytes * parity;
        load_1k_to_lds(a.K + off, voff0, set + 2048);
        load_1k_to_lds(a.Q + off, qoff, set + 4096);
        load_1k_to_lds(a.K + off, voff1, set + 3072);
        load_1k_to_lds(a.V + off, voff0, set);
        load_1k_to_lds(a.V + off, voff1, set + 1024);
    };

    // ---- accumulator input of the score product: bias (or 0) + 2^30, excluded / beyond the sequence: -2^29 + 2^30
    v16i cb[2];
    auto load_slice = [&](int s_idx) {
        if (PLAIN) {
            // Plain [N,N] layout: every lane reads its own row, 8 loads of four columns that each touch 32 rows'
            // lines; but once per run and slice, not once per pair.  (Buffer loads over the slice: one lane
            // offset for all of them, and dwords past the last row read 0 instead of leaving the tensor.
            // Rows need not start on 16 bytes: a load of four dwords asks for dword alignment only.)
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(a.bias + (size_t)s_idx * N * N), 0, 4 * N * N, 0x00020000);
            const int lane_off = 4 * (min(row, N - 1) * N + 4 * g);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int a4 = 0; a4 < 4; ++a4) {
                    const auto w = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off, 4 * (32 * kb + 8 * a4), 0);
#pragma unroll
                    for (int b = 0; b < 4; ++b) cb[kb][4 * a4 + b] = (int)w[b];
                }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    cb[kb][v] = (32 * kb + 8 * (v >> 2) + 4 * g + (v & 3) < N ? max(cb[kb][v], kWinExcluded) : kWinExcluded) + kAccBias;
        } else if (has_bias) {
            const int nb = (N + 31) / 32;                               // 2
            const int32_t* base = a.bias + (((size_t)s_idx * nb + half) * nb) * 1024 + 4 * lane;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int a4 = 0; a4 < 4; ++a4) {
                    const v4i w = *(const v4i*)(base + kb * 1024 + a4 * 256);
#pragma unroll
                    for (int b = 0; b < 4; ++b) cb[kb][4 * a4 + b] = max(w[b], kWinExcluded) + kAccBias;
                }
        } else {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    cb[kb][v] = (32 * kb + 8 * (v >> 2) + 4 * g + (v & 3) < N ? 0 : kWinExcluded) + kAccBias;
        }
    };

    // ---- the run.  Loads of a pair are issued one pair ahead; the output of a pair is stored one
    //      pair late, right after the only wait of the iteration, so that neither the loads nor the
    //      store are waited for while they are young.  Pairs of one bias slice form the inner loop:
    //      the accumulator input is invariant there.
    if (late) {
        table_in_place();
        if (PLAIN)
            for (int k = 0; k < (wave >> 2); ++k) __builtin_amdgcn_s_sleep(3);
    }
    issue_loads(p, 0);
    if (!late) table_in_place();
    int parity = 0;
    v4i o_prev = v4i{0, 0, 0, 0};
    size_t o_prev_off = 0;
    bool have_prev = false;
    const unsigned o_lane = (unsigned)(row * D + 16 * g);
    int t = t0;
    auto run_slice = [&] {
        const int t_end = min(t1, t + order.left_in_slice(p));       // pairs of this slice from here on
        for (; t < t_end; ++t) {
            // everything in flight belongs to this pair (or is the store of the one before the last)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const size_t o_off = (size_t)order.pair_index(p) * pair_bytes;
            order.advance(p);
            if (t + 1 < t1) issue_loads(p, parity ^ 1);
            if (have_prev && row < N) *(v4i*)(a.O + o_prev_off + o_lane) = o_prev;

            const int set = wbuf + kWinSetBytes * parity;
            o_prev = win_half<XM>(set + 4096 + op_lane, set + 2048 + op_lane, set + v_lane, cb, hc, c, a.out_round != 0, [] {});
            o_prev_off = o_off;
            have_prev = true;
            parity ^= 1;
        }
    };
    // (Two places that load a plain bias: in one, inside the loop, what every slice has in common is computed ahead of the first loads, 768 pairs
    // of 49 tokens 4.56 us a call against 4.31, 3072 of 64 9.40 and 9.12.  A packed one has little of that and is better off with the shorter
    // code: 2304 of 49 6.77 against 7.25, 3072 7.42 and 7.77.)
    if (PLAIN) {
        load_slice(p.s_idx);
        for (;;) {
            run_slice();
            if (t >= t1) break;
            load_slice(p.s_idx);
        }
    } else {
        while (t < t1) {
            load_slice(p.s_idx);
            run_slice();
        }
    }
    if (have_prev && row < N) *(v4i*)(a.O + o_prev_off + o_lane) = o_prev;
}

// ---- the same from float32 tensors and a bias in real units (dynamic quantisation)
//
// Replaces, after the abs-max pass, the quantising kernel, the one that converts the bias and the attention: the
// tensors are read once more and nothing but the output is written.  Bound by that read (5.8 TB/s at 12288
// pairs of 49 tokens).  Whole call, abs-max included: 12288 pairs 110.7 -> 79.3 us, 6144 62.5 -> 42.3,
// 3072 34.2 -> 26.7, 768 19.0 -> 14.5, 192 15.9 -> 10.7.  Three runs with one tensor (6 to 8 KiB) in flight
// per quantising wavefront measured best: two tensors 80.3 us, three 85; four runs 80.5, two 80.8.
//
// A workgroup has up to kWinDynStreams runs of pairs.  To each belong two wavefronts that compute (one
// half of the query rows each, as above, but from K and V in common) and two that quantise, a pair's
// K, Q and V in turn, into a ring of kWinDynSets sets of LDS; so the reads go on while the first two
// compute, and neither kind holds the other's registers.  Before the first pair the computing wavefronts
// derive the constants (wavefront 0), build the weight table and convert the bias of their run's slice,
// while the ring fills.  Synchronisation: filled[set] counts the tensors in place (3 per use of the set),
// emptied[set] the wavefronts that have read a use (2).  A use of a set begins only when its last one is
// read by both, so neither counter can run ahead.  Those who quantise wait only for those who compute the use
// before the last kWinDynSets - 1 pairs, those who compute only for theirs: every wavefront reaches its exit.
typedef unsigned u32_a1 __attribute__((aligned(1)));

template <int XM>
__device__ __forceinline__ void win_dyn_compute(const QflashLaunchArgs& a, const QflashHeadConsts& hc, double unit, const WinOrder& order,
                                                int t0, int t1, int half, int ring, int filled, int emptied) {
    constexpr int D = 32;
    round_down();                  // (single precision only: the bias is converted in double precision)
    const int N = a.N;
    const int lane = threadIdx.x & 63, g = lane >> 5, li = lane & 31;
    const int row = 32 * half + li;
    const ExpConst<> c = make_exp_const(hc);
    const int op_lane = 32 * li + 16 * g, v_lane = win_v_lane(lane);
    const double inv = 1.0 / unit;
    v16i cb[2];
    auto load_slice = [&](int s_idx) {
        // (all loads first.  Bias: as the plain bias above.  Mask: four bytes at a time, the last ones of a row from
        // four columns before its end, shifted)
        const size_t slice = (size_t)s_idx * N * N;
        const int first = min(row, N - 1) * N, col_l = 4 * g;
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((const float*)a.bias + (a.bias ? slice : 0)), 0, a.bias ? 4 * N * N : 0, 0x00020000);
        v4f x[8];
        unsigned mk[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < 8; ++w) x[w] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc, 4 * (first + col_l) + 32 * w, 0, 0));
        if (a.dyn_mask) {
            const uint8_t* m = a.dyn_mask + slice;
#pragma unroll
            for (int w = 0; w < 8; ++w) mk[w] = *(const u32_a1*)(m + first + min(col_l + 8 * w, N - 4));
#pragma unroll
            for (int w = 0; w < 8; ++w) mk[w] >>= 8 * min(max(col_l + 8 * w - (N - 4), 0), 3);
        }
#pragma unroll
        for (int w = 0; w < 8; ++w)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                cb[w >> 2][4 * (w & 3) + b] =
                    (col_l + 8 * w + b < N && (mk[w] >> (8 * b) & 0xffu) == 0 ? bias_word(x[w][b], unit, inv) : kWinExcluded) + kAccBias;
    };
    WinPair p = order.at(t0);
    int set = 0, use = 0;                    // set of the ring and how often it has been used before
    for (int t = t0; t < t1;) {
        load_slice(p.s_idx);
        const int t_end = min(t1, t + order.left_in_slice(p));
        for (; t < t_end; ++t) {
            const size_t o_off = (size_t)order.pair_index(p) * ((size_t)N * D);
            order.advance(p);
            wait_count(filled + 4 * set, 3 * (use + 1));
            const int s = ring + kWinDynSetBytes * set;
            const v4i o = win_half<XM>(s + 4096 + 1024 * half + op_lane, s + 2048 + op_lane, s + v_lane, cb, hc, c, a.out_round != 0,
                                       [&] { if (lane == 0) count_up(emptied + 4 * set); });
            if (row < N) *(v4i*)(a.O + o_off + (unsigned)(row * D + 16 * g)) = o;
            if (++set == kWinDynSets) { set = 0; ++use; }
        }
    }
}

__global__ __launch_bounds__(256 * kWinDynStreams) void qflash_fwd_win_dyn(const QflashLaunchArgs a) {
    constexpr int D = 32;
    constexpr int kDepth = 1;                     // tensors in flight per quantising wavefront
    const int N = a.N;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int S = a.win_streams;
    const int lds0 = (int)(size_t)(lds_void)smem_win;
    const int ring0 = lds0 + a.win_table_lds;
    // after the rings: [stream][set] filled, [stream][set] emptied, constants ready, table ready, constants
    const int cnt = ring0 + S * kWinDynSets * kWinDynSetBytes;
    const int hc_ready = cnt + 8 * S * kWinDynSets, table_ready = hc_ready + 4, hc_base = hc_ready + 8;
    for (int t = threadIdx.x; t < 2 * S * kWinDynSets + 2; t += blockDim.x) *(lds_int*)(size_t)(cnt + 4 * t) = 0;
    __syncthreads();

    const bool quantises = wave >= 2 * S;
    const int stream = (wave >> 1) - (quantises ? S : 0), sub = wave & 1;
    const int T = a.B * a.H;
    const int t0 = (blockIdx.x * S + stream) * a.win_chunk, t1 = min(t0 + a.win_chunk, T);
    const int ring = ring0 + stream * kWinDynSets * kWinDynSetBytes;
    const int filled = cnt + 4 * kWinDynSets * stream, emptied = filled + 4 * kWinDynSets * S;
    const WinOrder order(a, a.bias != nullptr || a.dyn_mask != nullptr);
    PartialMaxima pm;
    pm.load(a);

    if (quantises) {
        if (t0 >= t1) return;
        // item x of the run: tensor x % 3 (K, Q, V) of pair x / 3; this wavefront takes every second
        WinPair p = order.at(t0);
        int t = t0, tensor = sub, set = 0, use = 0;
        struct Item { int tensor, set, use; };           // tensor < 0: none
        v4f buf[kDepth][8];
        Item it[kDepth];
        auto issue = [&](int s) {
            it[s].tensor = t < t1 ? tensor : -1;
            it[s].set = set;
            it[s].use = use;
            const float* base = (const float*)(tensor == 0 ? a.K : tensor == 1 ? a.Q : a.V) + (size_t)order.pair_index(p) * N * D;
            // (rows beyond the sequence, and tensors beyond the run, read as zero)
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, t < t1 ? 4 * N * D : 0, 0x00020000);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                buf[s][u] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc, 16 * lane + 1024 * u, 0, 0));
            tensor += 2;
            if (tensor >= 3) {
                tensor -= 3;
                ++t;
                order.advance(p);
                if (++set == kWinDynSets) { set = 0; ++use; }
            }
        };
#pragma unroll
        for (int s = 0; s < kDepth; ++s) issue(s);
        const float r[3] = {pm.factor(1), pm.factor(0), pm.factor(2)};       // K, Q, V
        // (no way out of the middle of a trip: the compiler would have every trip wait for all its loads)
        while (it[0].tensor >= 0) {
#pragma unroll
            for (int s = 0; s < kDepth; ++s) {
                const Item x = it[s];
                const float rr = x.tensor == 0 ? r[0] : x.tensor == 1 ? r[1] : r[2];
                int packed[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) packed[u] = quantise4(buf[s][u], rr);
                // (converted before the registers are loaded again, not in the branch below)
                asm volatile("" : "+v"(packed[0]), "+v"(packed[1]), "+v"(packed[2]), "+v"(packed[3]), "+v"(packed[4]), "+v"(packed[5]),
                                  "+v"(packed[6]), "+v"(packed[7]));
                issue(s);
                if (x.tensor >= 0) {
                    wait_count(emptied + 4 * x.set, 2 * x.use);
                    const int dst = ring + kWinDynSetBytes * x.set + (x.tensor == 0 ? 2048 : x.tensor == 1 ? 4096 : 0) + 4 * lane;
#pragma unroll
                    for (int u = 0; u < 8; ++u) *(lds_int*)(size_t)(dst + 256 * u) = packed[u];
                    // (the LDS serves a wavefront's requests in order: the count is seen after the bytes)
                    if (lane == 0) count_up(filled + 4 * x.set);
                }
            }
        }
        return;
    }

    if (wave == 0) {
        const float am[3] = {pm.maximum(0), pm.maximum(1), pm.maximum(2)};
        if (lane == 0) {
            derive_to_lds(a, am, hc_base);
            count_up(hc_ready);
        }
    }
    wait_count(hc_ready, 1);
    const QflashHeadConsts hc = consts_from_lds(hc_base);
    const double unit = unit_from_lds(hc_base);
    if (hc.lut_bytes > 0) {
        table_to_lds(hc, lds0, wave, 2 * S);
        if (lane == 0) count_up(table_ready);
        wait_count(table_ready, 2 * S);
        win_dyn_compute<kExpTable>(a, hc, unit, order, t0, t1, sub, ring, filled, emptied);
    } else {
        win_dyn_compute<kExpShift>(a, hc, unit, order, t0, t1, sub, ring, filled, emptied);
    }
}

// PLAIN: a bias in the plain [N,N] layout; else a packed one or none.
template <int XM, bool PLAIN>
__global__ __launch_bounds__(1024) void qflash_fwd_win(const QflashLaunchArgs a) {
    if constexpr (XM == kExpAuto) {
        if (head_consts(a, 0).lut_bytes > 0) win_body<kExpTable, PLAIN>(a);
        else win_body<kExpShift, PLAIN>(a);
    } else {
        win_body<XM, PLAIN>(a);
    }
}

template <int XM, bool PLAIN>
int launch_win(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    return qflash_launch_kernel<qflash_fwd_win<XM, PLAIN>>(a, (unsigned)a.win_groups, (unsigned)(128 * a.win_streams), lds, lds_limit, st);
}

template <bool PLAIN>
int launch_mode(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    if (a.exp_mode == kExpTable) return launch_win<kExpTable, PLAIN>(a, lds, lds_limit, st);
    if (a.exp_mode == kExpShift0) return launch_win<kExpShift0, PLAIN>(a, lds, lds_limit, st);
    return launch_win<kExpShift, PLAIN>(a, lds, lds_limit, st);
}

}  // namespace

int qflash_launch_fwd_win(const QflashKernelArgs& a, int lds_limit, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    // everything the kernel's indexing assumes, checked once more where it is launched
    if (!a.win_mode || a.N <= 32 || a.N > 64 || a.win_streams < 1 || a.win_streams > 8 || a.win_chunk < 1 || a.win_groups < 1)
        return (int)hipErrorInvalidValue;
    if ((long long)a.win_groups * a.win_streams * a.win_chunk < (long long)a.B * a.H) return (int)hipErrorInvalidValue;
    if ((a.bias || (a.dyn_partial && a.dyn_mask)) && (a.bias_B < 1 || a.bias_H < 1 || a.B % a.bias_B != 0 || a.H % a.bias_H != 0))
        return (int)hipErrorInvalidValue;
    if (a.per_head || a.qmax) return (int)hipErrorInvalidValue;
    if (a.dyn_partial) {
        const size_t lds = qflash_win_dyn_lds_bytes(a.win_streams, a.win_table_lds);
        if (a.win_streams > kWinDynStreams || a.lut_bytes_max > a.win_table_lds || a.dyn_partials > 256 || lds > (size_t)lds_limit)
            return (int)hipErrorInvalidValue;
        return qflash_launch_kernel<qflash_fwd_win_dyn>(a, (unsigned)a.win_groups, (unsigned)(256 * a.win_streams), lds, lds_limit, st);
    }
    const bool table = a.exp_mode == kExpTable || a.exp_mode == kExpAuto;
    if (table && a.lut_bytes_max > a.win_table_lds) return (int)hipErrorInvalidValue;
    const size_t lds = qflash_win_lds_bytes(a.win_streams, table ? a.win_table_lds : 0);
    if (lds > (size_t)lds_limit) return (int)hipErrorInvalidValue;
    // (constants made on the GPU come without a bias: with one the kernel above makes them itself)
    if (a.exp_mode == kExpAuto) return a.bias ? (int)hipErrorInvalidValue : launch_win<kExpAuto, false>(a, lds, lds_limit, st);
    return a.bias && !a.bias_packed ? launch_mode<true>(a, lds, lds_limit, st) : launch_mode<false>(a, lds, lds_limit, st);
}
