// gfx950 kernel of the integer-only fused attention forward pass (Algorithm 1) for short sequences
// with 64 features per head and no bias: one workgroup fills a whole compute unit.
//
// A workgroup of up to 16 wavefronts takes `cu_heads` consecutive (batch, head) pairs.  Q, K and V
// of all of them, plus the weight table, go to LDS once, by direct global-to-LDS loads: no staging
// registers, no vector instructions besides a few address computations, no LDS write instructions.
// The tensors sit in LDS row-major as in memory (64-byte rows, the 16-byte pieces of a row permuted
// by the row number so that operand reads are free of bank conflicts); the transposed operand of the
// second product is read with the transposing 8-bit LDS read (see qflash_tile.h).  The unit of work
// is one block of 32 query rows of one pair.  Each wavefront starts with the unit of its own index
// and then takes further units from a counter in LDS, so wavefronts run at their own pace: there is
// no barrier after the start.
//
// Synchronisation.  The loads of a pair are issued by the wavefronts whose first unit belongs to it
// (pairs without such wavefronts: by the last group that has some), in the order of need.  Loads
// complete in order, so a wavefront knows from its own load counter (vmcnt) when its share of a
// tile has landed; it then adds 1 to the counter of (pair, tile) in LDS, and a wavefront may touch
// the data of a tile once that counter has reached the size of the issuing group.  Every wait in
// the kernel is for loads that were issued unconditionally before it and for counters that other
// wavefronts raise without waiting for anybody but their own loads, so every wavefront reaches its
// exit.
//
// 64 features, 768 pairs of 197 tokens: 16.9 -> 15.6 us with ScaleRelease, packing and normalisation on the float units
// (qflash_tile.h), per head 21.7 -> 18.9.  What is left: LDS 9 us of look-ups and operand reads, vector issue 7, 3 us until
// every wavefront has data, five units for sixteen wavefronts at the end.
//
// A workgroup requests its first tile when a wavefront has found out what to request; the quotients it needs for that are made with reciprocals
// from the host (or counted up), not by division: 768 pairs of 197 tokens 15.55 -> 15.2 us a call, per head, where two were of 64 bits, 18.9 -> 18.5
// and 21.0 -> 19.7 with tiles of 128, 180 of 256 from the static entry point 9.55 -> 9.35.
//
// KV tiles of 128: more than 128 registers leave three wavefronts to a SIMD, so workgroups are at most twelve; still ahead of
// the resident kernel (768 pairs of 197 tokens 22.8 -> 18.6 us, 480 of 256 19.4 -> 15.0, 720 of 130 16.8 -> 12.4).
//
// QF_TRACE (never defined in the library build) adds per-wavefront timestamps for timeline studies.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "qflash_counters.h"
#include "qflash_derive_device.h"
#include "qflash_launch.h"
#include "qflash_tile.h"

// (M0 is written by the direct loads below and declared as clobbered; the compiler's remark that it
// reserves the register for itself does not apply to a kernel that uses no other M0 instruction)
#pragma clang diagnostic ignored "-Winline-asm"

namespace {

extern __shared__ __align__(1024) int8_t smem_cu[];

template <int XM> struct WeightMode { static constexpr int value = XM; };

#ifdef QF_TRACE
// timestamps go to LDS (an instruction the compiler does not count, like the counters) and are copied out at the end
#define QF_T(K_) do { if ((K_) < 16) { const unsigned long long t_ = __builtin_amdgcn_s_memrealtime(); \
    const int ta_ = trace_base + 8 * (16 * wave + (K_)); \
    asm volatile("ds_write_b64 %0, %1" :: "v"(ta_), "v"(t_) : "memory"); } } while (0)
#else
#define QF_T(K_) do {} while (0)
#endif

// The units of a workgroup, from unit u0 of this wavefront on.  ready(pair, tile, first tile of the unit, first unit of the
// wavefront) returns when the tile (and what goes with the first one of a unit) is in LDS; next_unit: LDS
// address of the counter; PH: hc0 are the constants of the table's head, otherwise of the launch.
template <int XM, bool PH, int BC, class Args, class Ready, class PairOf, class HeadOf>
__device__ __forceinline__ void cu_units(const Args& a, const QflashHeadConsts& hc0, int table_head, int u0, int units,
                                         int nblk, int kv_base, int slot, int next_unit, int wave, int trace_base,
                                         Ready ready, PairOf pair_of, HeadOf head_of) {
    constexpr int D = 64;
    round_down();
    const int N = a.N;
    const int lane = threadIdx.x & 63, g = lane >> 5, li = lane & 31;
    const SwizzledLane sl = swizzled_lane_offsets<D>(lane);
    const ExpConst<> c0 = make_exp_const<XM != kExpTable || PH>(hc0);
    const int n_tiles = (N + BC - 1) / BC;
    [[maybe_unused]] int tk = 3;

    // Units: wavefront w starts with unit w; all further ones come from the counter.
    bool first_unit = true;
    int u = u0;
    while (u < units) {
        // (the sequence length through an opaque copy: the compiler would otherwise evaluate every
        // "is this group of keys inside the sequence" test of the ragged tile once, ahead of the loop,
        // and keep the answers in more scalar registers than there are)
        int N_ = N;
        asm volatile("" : "+s"(N_));
        // (likewise the lane's half: the key indices of the ragged tile derive from it, two dozen
        // registers' worth if they are prepared ahead of the loop)
        int g_ = g;
        asm volatile("" : "+v"(g_));
        const int n_full = N_ / BC, rem = N_ - n_full * BC;
        const int h = qflash_small_quotient(u, a.cu_inv_nblk), blk = u - h * nblk;
        const int Kb = kv_base + 3 * h * slot, Vb = Kb + slot, Qb = Vb + slot;
        const int row0 = 32 * blk, i = row0 + li;
        RowState<D> st;
        st.l = 0;
        v4i qreg[2];
        QflashHeadConsts hc = hc0;
        if constexpr (PH) hc = own_head_consts(a, head_of(h));
        const ExpConst<> c = PH ? make_exp_const(hc) : c0;
#define QF_TILE(FULL_, FIRST_, J_, NV_, NG_)                                                               \
        ready(h, J_, FIRST_, first_unit);                                                                  \
        if (FIRST_) QF_T(tk);                                                                              \
        if (FIRST_) {                                                                                      \
            _Pragma("unroll") for (int s = 0; s < 2; ++s)                                                  \
                qreg[s] = *(lds_v4i*)(size_t)(Qb + row0 * D + (sl.k_off ^ (32 * s)));                      \
        }                                                                                                  \
        process_tile<D, BC, kBiasNone, UM, UM == kExpTable, FULL_, FIRST_, kLaySwizzled, NG_, false, kReleaseFloat>(                 \
            st, qreg, nullptr, 0, nullptr, 0, NV_, hc.lut_xp, nullptr, nullptr, c, hc.a_mul, li, g_,      \
            Kb + D * BC * (J_) + sl.k_off, Vb + D * BC * (J_) + sl.v_off);                                 \
        if (tk == 6) QF_T(9 + (J_))
        // the ragged tile, with its number of groups of 8 keys as a compile-time constant (tiles of 64)
#define QF_RAGGED(FIRST_, J_)                                                                              \
        if constexpr (BC == 128) { QF_TILE(false, FIRST_, J_, rem, 0); }                                   \
        else switch ((rem + 7) >> 3) {                                                                     \
            case 1: { QF_TILE(false, FIRST_, J_, rem, 1); } break;                                         \
            case 2: { QF_TILE(false, FIRST_, J_, rem, 2); } break;                                         \
            case 3: { QF_TILE(false, FIRST_, J_, rem, 3); } break;                                         \
            case 4: { QF_TILE(false, FIRST_, J_, rem, 4); } break;                                         \
            case 5: { QF_TILE(false, FIRST_, J_, rem, 5); } break;                                         \
            case 6: { QF_TILE(false, FIRST_, J_, rem, 6); } break;                                         \
            case 7: { QF_TILE(false, FIRST_, J_, rem, 7); } break;                                         \
            default: { QF_TILE(false, FIRST_, J_, rem, 8); } break;                                        \
        }
        auto walk = [&](auto mode) {
            constexpr int UM = decltype(mode)::value;          // weight mode of this unit
            st.m = UM == kExpTable ? (int)((unsigned)kMInit + (unsigned)kAccBias) : kMInit;
            if (n_full > 0) {
                QF_TILE(true, true, 0, BC, 0);
                for (int j = 1; j < n_full; ++j) { QF_TILE(true, false, j, BC, 0); }
                if (rem > 0) { QF_RAGGED(false, n_full) }
            } else {
                QF_RAGGED(true, 0)
            }
        };
        if constexpr (PH && XM == kExpTable) {
            if (head_of(h) == table_head) walk(WeightMode<kExpTable>{});
            else walk(WeightMode<kExpShift>{});
        } else {
            walk(WeightMode<XM>{});
        }
#undef QF_RAGGED
#undef QF_TILE
        first_unit = false;
        QF_T(tk + 1);
        if (i < N) {
            // (uniform base plus a 32-bit lane offset made here: a per-lane 64-bit pointer prepared ahead of
            // the unit loop would be held in registers across all the tile code, or spilled)
            v4i w[2];
            if (a.out_round == 0) float_normalise_words<D, kAccOffset>(st, w);
            else normalise_words<D, 16, kAccOffset>(st, true, w);
            int8_t* Ob = a.O + (size_t)pair_of(h) * N * D;
            unsigned o_lane = (unsigned)(i * D + g * (D / 2));
            asm volatile("" : "+v"(o_lane));
            *(v4i*)(Ob + o_lane) = w[0];
            *(v4i*)(Ob + o_lane + 16) = w[1];
        }
        // next unit
        int nxt = 0;
        if (lane == 0) nxt = __hip_atomic_fetch_add((lds_int*)(size_t)(next_unit), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        u = __builtin_amdgcn_readfirstlane(nxt);
        QF_T(tk + 2);
        tk += 3;
    }
    QF_T(15);
}

// PH: one set of constants per head.  The pairs are then dealt out so that every workgroup gets its share of
// those with a table and of those without, the former one head after the other: a workgroup stages
// the table of its first pair's head, and a unit of a pair of another head computes its weights.
template <bool PH> using CuArgs = std::conditional_t<PH, QflashKernelArgs, QflashLaunchArgs>;

template <int XM, bool PH, int BC>
__device__ __forceinline__ void cu_body(const CuArgs<PH>& a) {
    constexpr int D = 64;
    const int N = a.N;
    const int rows16 = (N + 15) & ~15;
    const int slot = rows16 * D;                    // LDS bytes of one tensor of one pair
    const int nblk = (N + 31) >> 5;                 // units per pair
    const int hpw = a.cu_heads;
    const int head0 = blockIdx.x * hpw;
    const int n_heads = min(hpw, a.B * a.H - head0);
    // PH: lane h < n_heads holds pair and head of slot h.  Slots [p0, p0 + n_heads) of the launch: T of the P
    // pairs have a table, so slot position p stands behind p T / P of them (rounded down).
    [[maybe_unused]] int pair_l = 0, head_l = 0, table_head = -1;
    if constexpr (PH) {
        const int P = a.B * a.H, T = a.cu_table_heads * a.B;
        unsigned rest, batch;
        const int t0 = (int)qflash_divide((unsigned)head0 * (unsigned)T, (unsigned)P, a.cu_inv_pairs, &rest);
        const int n_t = (int)qflash_divide((unsigned)(head0 + n_heads) * (unsigned)T, (unsigned)P, a.cu_inv_pairs, &rest) - t0;
        const int h = min((int)(threadIdx.x & 63), n_heads - 1);
        const int x = h < n_t ? t0 + h : T + (head0 - t0) + (h - n_t);          // position in head order
        head_l = a.cu_order[qflash_divide((unsigned)x, (unsigned)a.B, a.cu_inv_b, &batch)];
        pair_l = (int)batch * a.H + head_l;
        if (n_t > 0) table_head = __builtin_amdgcn_readfirstlane(head_l);
    }
    auto pair_of = [&](int h) { return PH ? __builtin_amdgcn_readlane(pair_l, h) : head0 + h; };
    const int units = n_heads * nblk;
    const int n_waves = min((int)(blockDim.x >> 6), units);   // the last workgroup may have fewer pairs: extra wavefronts leave
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // LDS map (dynamic LDS is the only LDS of this kernel, so it starts at address 0 and the index
    // into the weight table is its address): [table][pair 0: K, V, Q][pair 1: ...] ... [1 KiB that
    // reads of the 32-row blocks past the last 16-row block may touch][counters]
    const int lds0 = (int)(size_t)(lds_void)smem_cu;          // 0: checked by the host before the first launch
    const int tbytes = XM == kExpTable ? a.cu_table_lds : 0;
    const int kv_base = lds0 + tbytes;
    // counters: [pair][tile]: wavefronts of the group whose loads for that tile have landed; [4 * hpw]: next unit
    const int cnt_base = kv_base + hpw * 3 * slot + 1024;
#ifdef QF_TRACE
    const int trace_base = cnt_base + 4 * (5 * hpw + 1) + 8;
    for (int t = threadIdx.x; t < 512; t += blockDim.x) *(lds_int*)(size_t)(trace_base + 4 * t) = 0;
    __syncthreads();
#endif
    QF_T(0);
    for (int t = threadIdx.x; t <= 5 * hpw; t += blockDim.x) *(lds_int*)(size_t)(cnt_base + 4 * t) = t == 4 * hpw ? n_waves : 0;
    __syncthreads();
    if (wave >= n_waves) return;
    QF_T(1);

    // constants of the launch; PH: of the table's head, each unit then takes those of its own
    QflashHeadConsts hc0;
    if constexpr (PH) hc0 = own_head_consts(a, max(table_head, 0));
    else hc0 = head_consts(a, 0);

    // ---- loop-invariant registers
    const int nb16 = rows16 >> 4;                   // 1 KiB loads per tensor of a pair
    const int nt = XM == kExpTable && (!PH || table_head >= 0) ? (hc0.lut_bytes + 1023) >> 10 : 0;   // 1 KiB loads of the table

    // ---- the loads.  The wavefronts whose first unit belongs to pair g (its group) share the loads of
    //      that pair: member m of a group of n takes the pieces of the table (group 0 only), the 16-row
    //      blocks of Q and the blocks of K and V (numbered 2 * block + (V ? 1 : 0), i.e. tile by tile)
    //      whose number is m modulo n, and issues them at once in that order, which is the order of
    //      need.  Groups start one after the other (a short sleep), so that the memory system sees
    //      the requests of pair 0 first.  Pairs beyond the last group are taken by that group as
    //      well, after its own; they are only needed in the second round.
    //      A wavefront waits for its loads of the first tile right after issuing them and adds 1 to
    //      the counter of (pair, tile 0); before the second tile of its first unit it waits for all its
    //      loads (they have had a whole tile's time) and adds 1 to the counters of all other tiles.
    //      Before any tile of any unit a wavefront waits until the counter of (pair, tile) has reached
    //      the size of the group.
    const int last_group = qflash_small_quotient(n_waves - 1, a.cu_inv_nblk);
    const int my_group = qflash_small_quotient(wave, a.cu_inv_nblk);
    const int group_size = min(nblk, n_waves - my_group * nblk);
    const int member = wave - my_group * nblk;
    const int n_extra = my_group == last_group ? n_heads - 1 - my_group : 0;     // whole pairs
    // A last group of fewer wavefronts than the others gets help with the first tile of its pair from
    // group 0 (whose wavefronts issue their share after their own loads and report it with their
    // other late loads, before the second tile of their first unit).
    const int last_size = n_waves - last_group * nblk;
    const bool small_last = last_group > 0 && last_size < nblk;
    const bool helper = small_last && my_group == 0, helped = small_last && my_group == last_group;
    {
        // Lane part of the address inside a 16-row block: row lane / 4, 16-byte piece (lane % 4)
        // permuted by the row.  The last block of a tensor may reach beyond the sequence: its rows are
        // clamped to the last row (what lands in the padding rows is never used).
        const int lrow = lane >> 2, piece = ((lane & 3) ^ ((lane >> 4) & 3)) << 4;
        const int off_norm = lrow * D + piece;
        const int off_last = (min(16 * (nb16 - 1) + lrow, N - 1) - 16 * (nb16 - 1)) * D + piece;
        // First tile of the own pair (and the table).  The other groups start when the first tile of
        // group 0 has landed: the memory system shares its bandwidth evenly between whatever is in
        // flight, so this is what lets group 0 start computing while the others are still loading.
        if (my_group > 0) wait_count(cnt_base, nblk);
        if (XM == kExpTable && my_group == 0)
            for (int it = member; it < nt; it += group_size)
                load_1k_to_lds((const int8_t*)hc0.lut + 1024 * it, 16 * lane, lds0 + 1024 * it);
        const int x0 = min(BC / 8, 2 * nb16);                       // K/V block numbers of the first tile
        auto load_q = [&](int h, int mi, int np) {
            const size_t head_off = (size_t)pair_of(h) * N * D;
            for (int b = mi; b < nb16; b += np)
                load_1k_to_lds(a.Q + head_off + 1024 * b, b == nb16 - 1 ? off_last : off_norm,
                               kv_base + (3 * h + 2) * slot + 1024 * b);
        };
        auto load_kv = [&](int h, int x_lo, int x_hi, int mi, int np) {
            const size_t head_off = (size_t)pair_of(h) * N * D;
            int x = mi;                                             // (mi < np; counted up: a division takes longer)
            while (x < x_lo) x += np;
            for (; x < x_hi; x += np) {
                const int b = x >> 1;
                load_1k_to_lds(((x & 1) ? a.V : a.K) + head_off + 1024 * b, b == nb16 - 1 ? off_last : off_norm,
                               kv_base + (3 * h + (x & 1)) * slot + 1024 * b);
            }
        };
        // (a last group of few wavefronts shares the first tile of its pair with the group before it)
        const int s0_np = helped ? group_size + nblk : group_size, s0_mi = helped ? nblk + member : member;
        load_q(my_group, s0_mi, s0_np);
        load_kv(my_group, 0, x0, s0_mi, s0_np);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) count_up(cnt_base + 4 * (4 * my_group));
        // the other tiles, then further pairs, then the share of the next group's first tile
        load_kv(my_group, x0, 2 * nb16, member, group_size);
        for (int e = 1; e <= n_extra; ++e) {
            load_q(my_group + e, member, group_size);
            load_kv(my_group + e, 0, 2 * nb16, member, group_size);
        }
        if (helper) {
            load_q(last_group, member, nblk + last_size);
            load_kv(last_group, 0, x0, member, nblk + last_size);
        }
    }
    QF_T(2);
    const int n_tiles = (N + BC - 1) / BC;
    auto ready = [&](int h, int j, bool first, bool first_unit) {
        if (first_unit && j == (n_tiles > 1 ? 1 : 0)) {
            // second tile of the first unit (or its only one): all own loads have had a tile's time
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) {
                if (helper) count_up(cnt_base + 4 * (4 * last_group));
                for (int s = 1; s < n_tiles; ++s) count_up(cnt_base + 4 * (4 * my_group + s));
                for (int e = my_group + 1; e <= my_group + n_extra; ++e)
                    for (int s = 0; s < n_tiles; ++s) count_up(cnt_base + 4 * (4 * e + s));
            }
        }
        if (first && XM == kExpTable && h != 0) wait_count(cnt_base, min(nblk, n_waves));
        const int owner = min(h, last_group);
        const int target = min(nblk, n_waves - owner * nblk);
        wait_count(cnt_base + 4 * (4 * h + j), j == 0 && small_last && h == last_group ? target + nblk : target);
    };
#ifndef QF_TRACE
    const int trace_base = 0;
#endif
    cu_units<XM, PH, BC>(a, hc0, table_head, wave, units, nblk, kv_base, slot, cnt_base + 4 * 4 * hpw, wave, trace_base, ready,
                     pair_of, [&](int h) { return __builtin_amdgcn_readlane(head_l, h); });
#ifdef QF_TRACE
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (a.trace && lane < 16)
        a.trace[((size_t)blockIdx.x * 16 + wave) * 16 + lane] = *(const __attribute__((address_space(3))) unsigned long long*)(size_t)(trace_base + 8 * (16 * wave + lane));
#endif
}

template <int XM, bool PH, int BC>
__global__ __launch_bounds__(64 * qflash_cu_max_waves(BC)) void qflash_fwd_cu(const CuArgs<PH> a) {
    cu_body<XM, PH, BC>(a);
}

// ---- the same from float32 tensors (dynamic quantisation): the kernel quantises on the way into LDS
//
// After the abs-max pass the tensors are read once more and neither the int8 copies nor the constants
// travel through memory: 12 B read + 1 B written per element triple instead of 12 + 3 and 3 + 1 in two
// launches, and all but the last pair's attention runs while floats are still arriving.  Bound by that
// read (from the last-level cache where the tensors fit it).  Whole call, abs-max included: 768 pairs of 197
// tokens 64.8 -> 48.4 us, 384 35.6 -> 29.4, 480 of 256 52.5 -> 40.8, 2048 of 50 40.0 -> 29.9.
//
// Wavefront 0 derives the constants (double precision on one lane, 3 us); the others quantise the
// first pairs, 4 KiB of floats (16 rows) at a time with two pieces of loads in flight each (with one
// or two 48 us, with three or four 51).  Then the first `workers` wavefronts build the weight table
// in LDS and start on the units, while the others go on quantising pair after pair and join them at
// the end (8 workers: with 4 to 12 of the 16 within 3 %).  Nobody waits for anything but loads, the
// constants (wavefront 0 waits for no other) and the table and tiles that the former two lead to, so
// every wavefront reaches its exit.
constexpr int kCuDynWorkers = 8;      // at most: wavefronts that start on the units while the others quantise

template <int BC>
__global__ __launch_bounds__(64 * qflash_cu_max_waves(BC)) void qflash_fwd_cu_dyn(const QflashLaunchArgs a) {
    constexpr int D = 64, kTileBlocks = BC / 16, kWaves = qflash_cu_max_waves(BC);
    constexpr int kDepth = 2;                       // pieces in flight per wavefront
    const int N = a.N;
    const int nb16 = (N + 15) >> 4;                 // pieces per tensor of a pair
    const int slot = 16 * nb16 * D;
    const int nblk = (N + 31) >> 5;
    const int hpw = a.cu_heads;
    const int head0 = blockIdx.x * hpw;
    const int n_heads = min(hpw, a.B * a.H - head0);
    const int units = n_heads * nblk;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int early = min(n_heads, max(1, qflash_small_quotient(kCuDynWorkers, a.cu_inv_nblk)));     // pairs that everybody quantises first
    const int workers = min(early * nblk, kCuDynWorkers);

    // LDS map: as above, then [constants ready][wavefronts done with the table][the constants]
    const int lds0 = (int)(size_t)(lds_void)smem_cu;
    const int kv_base = lds0 + a.cu_table_lds;
    const int cnt_base = kv_base + hpw * 3 * slot + 1024;
    const int next_unit = cnt_base + 16 * hpw, hc_ready = next_unit + 4, table_ready = next_unit + 8, hc_base = next_unit + 12;
    for (int t = threadIdx.x; t < 4 * hpw + 3; t += blockDim.x) *(lds_int*)(size_t)(cnt_base + 4 * t) = t == 4 * hpw ? workers : 0;
    __syncthreads();

    PartialMaxima pm;
    pm.load(a);

    if (wave == 0) {
        const float am[3] = {pm.maximum(0), pm.maximum(1), pm.maximum(2)};
        if (lane == 0) {
            derive_to_lds(a, am, hc_base);
            count_up(hc_ready);
        }
    } else {
        // ---- pieces: index x of the launch's share -> pair x / per; inside a pair the blocks of Q, then
        //      those of K and V in turn
        const int per = 3 * nb16;
        struct Piece { int x, h, y; };               // h < 0: none left
        const int first_end = early * per, end = n_heads * per;
        auto place = [&](int x) {
            Piece p;
            p.x = x;
            p.h = x < end ? (int)__umulhi((unsigned)x, a.cu_inv_per) : -1;
            p.y = x - p.h * per;
            return p;
        };
        auto next = [&](int x) {
            if (x < first_end) {
                x += kWaves - 1;
                if (x >= first_end) x = wave >= workers ? first_end + wave - workers : end;
            } else {
                x += kWaves - workers;
            }
            return place(x);
        };
        v4f buf[kDepth][4];
        Piece pc[kDepth];
        // loads of a piece: lane l takes 16 bytes of row 4 u + l / 16; what lies beyond the sequence (or a
        // piece that does not exist) reads as zero
        auto issue = [&](int s) {
            const Piece p = pc[s];
            const int h = max(p.h, 0), z = p.y - nb16, b = z < 0 ? p.y : z >> 1;
            const float* base = (const float*)(z < 0 ? a.Q : (z & 1) ? a.V : a.K) + (size_t)(head0 + h) * N * D + 1024 * b;
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, p.h < 0 ? 0 : 4 * (N * D - 1024 * b), 0x00020000);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                buf[s][u] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc, 16 * lane + 1024 * u, 0, 0));
        };
        const int x0 = wave - 1;
        pc[0] = place(x0 < first_end ? x0 : wave >= workers ? first_end + wave - workers : end);
        issue(0);
#pragma unroll
        for (int s = 1; s < kDepth; ++s) { pc[s] = next(pc[s - 1].x); issue(s); }
        const float r[3] = {pm.factor(0), pm.factor(1), pm.factor(2)};
        // byte of row 4 u + lane / 16: the 16-byte pieces of a row are permuted by (row / 4) & 3 = u
        const int w_lane = 64 * (lane >> 4) + 16 * ((lane & 15) >> 2) + 4 * (lane & 3);
        // (no way out of the middle of a trip: the compiler would have every trip wait for all its loads)
        while (pc[0].h >= 0) {
#pragma unroll
            for (int s = 0; s < kDepth; ++s) {
                const Piece p = pc[s];
                const int z = p.y - nb16, b = z < 0 ? p.y : z >> 1;
                const float rr = z < 0 ? r[0] : (z & 1) ? r[2] : r[1];
                const int dst = kv_base + (3 * p.h + (z < 0 ? 2 : z & 1)) * slot + 1024 * b;
                int packed[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) packed[u] = quantise4(buf[s][u], rr);
                // (converted before the registers are loaded again, not in the branch below)
                asm volatile("" : "+v"(packed[0]), "+v"(packed[1]), "+v"(packed[2]), "+v"(packed[3]));
                pc[s] = next(pc[(s + kDepth - 1) % kDepth].x);
                issue(s);
                if (p.h >= 0) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) *(lds_int*)(size_t)(dst + (w_lane ^ (16 * u)) + 256 * u) = packed[u];
                    // (the LDS serves a wavefront's requests in order: the count is seen after the bytes)
                    if (lane == 0) count_up(cnt_base + 4 * (4 * p.h + (z < 0 ? 0 : b / kTileBlocks)));
                }
            }
        }
    }

    // ---- constants; the weight table
    wait_count(hc_ready, 1);
    const QflashHeadConsts hc = consts_from_lds(hc_base);
    if (wave < workers && hc.lut_bytes > 0) {
        table_to_lds(hc, lds0, wave, workers);
        if (lane == 0) count_up(table_ready);
    }
    int u0 = wave;
    if (wave >= workers) {
        int nxt = 0;
        if (lane == 0) nxt = __hip_atomic_fetch_add((lds_int*)(size_t)next_unit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        u0 = __builtin_amdgcn_readfirstlane(nxt);
    }
    auto ready = [&](int h, int j, bool first, bool first_unit) {
        if (first && first_unit && hc.lut_bytes > 0) wait_count(table_ready, workers);
        wait_count(cnt_base + 4 * (4 * h + j), 2 * (min(kTileBlocks * (j + 1), nb16) - kTileBlocks * j) + (j == 0 ? nb16 : 0));
    };
    auto pair_of = [&](int h) { return head0 + h; };
    auto head_of = [](int) { return 0; };
    if (hc.lut_bytes > 0)
        cu_units<kExpTable, false, BC>(a, hc, 0, u0, units, nblk, kv_base, slot, next_unit, wave, 0, ready, pair_of, head_of);
    else
        cu_units<kExpShift, false, BC>(a, hc, 0, u0, units, nblk, kv_base, slot, next_unit, wave, 0, ready, pair_of, head_of);
}

template <int XM, bool PH, int BC>
int launch_cu(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    return qflash_launch_kernel<qflash_fwd_cu<XM, PH, BC>>(a, (unsigned)a.cu_groups, (unsigned)(64 * a.cu_waves), lds, lds_limit, st);
}

template <int BC>
int launch_tile(const QflashKernelArgs& a, bool table, size_t lds, int lds_limit, hipStream_t st) {
    if (a.dyn_partial)
        return qflash_launch_kernel<qflash_fwd_cu_dyn<BC>>(a, (unsigned)a.cu_groups, 64 * qflash_cu_max_waves(BC), lds, lds_limit, st);
    if (a.per_head) {
        if (table) return launch_cu<kExpTable, true, BC>(a, lds, lds_limit, st);
        if (a.exp_mode == kExpShift0) return launch_cu<kExpShift0, true, BC>(a, lds, lds_limit, st);
        return launch_cu<kExpShift, true, BC>(a, lds, lds_limit, st);
    }
    if (table) return launch_cu<kExpTable, false, BC>(a, lds, lds_limit, st);
    if (a.exp_mode == kExpShift0) return launch_cu<kExpShift0, false, BC>(a, lds, lds_limit, st);
    return launch_cu<kExpShift, false, BC>(a, lds, lds_limit, st);
}

}  // namespace

int qflash_launch_fwd_cu(const QflashKernelArgs& a, int lds_limit, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (!a.cu_mode || a.cu_heads < 1 || a.cu_waves < 1 || a.cu_waves > qflash_cu_max_waves(a.kv_tile) || a.N > 256 || a.bias ||
        (a.kv_tile != 64 && a.kv_tile != 128))
        return (int)hipErrorInvalidValue;
    // (what qflash_small_quotient is exact for; products of two numbers of pairs, per head, in 32 bits)
    const long long nblk = (a.N + 31) / 32;
    if (a.cu_heads * nblk * nblk >= 65536 || (a.per_head && (long long)a.B * a.H >= 65536)) return (int)hipErrorInvalidValue;
    if (a.dyn_partial && (a.per_head || a.dyn_partials > 256)) return (int)hipErrorInvalidValue;
    if (!a.dyn_partial && a.hc_dev) return (int)hipErrorInvalidValue;
    if (a.per_head && (a.cu_table_heads < 0 || a.cu_table_heads > a.H || a.H > kQflashMaxParamHeads)) return (int)hipErrorInvalidValue;
    // (per-head constants, mode Auto: some heads have a table)
    const bool table = a.dyn_partial || a.exp_mode == kExpTable || (a.exp_mode == kExpAuto && a.per_head);
    if (table && a.lut_bytes_max > a.cu_table_lds) return (int)hipErrorInvalidValue;
    const size_t lds = qflash_cu_lds_bytes(a.N, a.cu_heads, table ? a.cu_table_lds : 0) + (a.dyn_partial ? kCuDynExtraLds : 0);
    if (lds > (size_t)lds_limit) return (int)hipErrorInvalidValue;
    return a.kv_tile == 64 ? launch_tile<64>(a, table, lds, lds_limit, st) : launch_tile<128>(a, table, lds, lds_limit, st);
}
