// gfx950 kernel of the integer-only fused attention forward pass (Algorithm 1) for long sequences
// without a bias: the ring fed by direct global-to-LDS loads.
//
// A workgroup of up to 8 wavefronts serves 32 query rows per wavefront of one (batch, head) pair and
// walks over all KV tiles of the pair.  LDS holds the weight table and three (64 features) or four slots, each
// of one tile of K or V.  The tiles arrive row-major as they lie in memory (16-byte pieces permuted by the row so
// that operand reads are free of bank conflicts), put there by `global_load_lds_dwordx4`; the K/Q operands are
// plain 16-byte LDS reads and the V^T operand is read with the transposing 8-bit LDS read (see qflash_tile.h).
// Compared with staging through registers (qflash_resident.h) there are no staging registers, no byte transposes
// in the vector ALU and no LDS write instructions: about a third of that kernel's vector instructions on these shapes.
//
// What bounds it (cycles at 2.2 GHz, per wavefront and KV tile of 64):
//   64 features, tiny table (256 pairs of 577 tokens, tiles of 64, 26.1 -> 20.4 us): in steady state (four times the
//     pairs) 770 cycles of a SIMD for 146 vector instructions and 8 matrix instructions of 32 cycles, during which hardly
//     any float instruction issues; a lone wavefront takes 2300.  5 of the 20 us are the start (first loads, 2 us) and the end.
//   64 features, tiles of 128 (384 pairs of 577, 39.1 -> 33.8 us): four wavefronts to a SIMD instead of three, as far
//     as registers (128) and LDS (three slots, not four: 35 KiB with the table) go; then the same.
//   32 features (64 pairs of 2100 tokens, 73.0 -> 59.7 us): LDS, 24 look-ups with 5.3 conflict cycles each, against the
//     eight computed weights in thirty-two on the vector units (MIXED of process_tile).
// 32 features against the streamed kernel that staged one tile at a time through registers and computed the weights:
// B*H = 64, N = 2100 145.6 -> 59.7 us with tiles of 64, 202 -> 65 us with tiles of 128.
//
// Synchronisation: the wavefronts share the loads of a tile (1 KiB pieces, dealt round robin), wait for their own (vmcnt)
// and then for the others at a barrier; see QF_RING_TILE.  Every wavefront of a workgroup executes every barrier, with
// or without query rows of its own.  (Three slots: V of a tile is requested behind the tile before it, when its place,
// the one of that tile's K, is free; requested at the start of its own tile the last, short one waited for it.)
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "qflash_launch.h"
#include "qflash_tile.h"

// (M0 is written by the direct loads below and declared as clobbered)
#pragma clang diagnostic ignored "-Winline-asm"

namespace {

extern __shared__ __align__(1024) int8_t smem_ring[];

// ScaleRelease: the float form, and beyond its range the integer form on the same accumulators.
template <bool QMAX>
constexpr int ring_release(bool in_range) { return QMAX ? kReleaseInt : in_range ? kReleaseFloat : kReleaseMoved; }

template <int V> struct RingInt { static constexpr int value = V; };

// Weight tables of 32 features from this size on: part of the weights is computed (MIXED of process_tile).
constexpr int kRingMixedBytes = 7 * 1024;

template <int D, int BC, int XM, bool QMAX, int MIXED = 0>
__device__ __forceinline__ void ring_body(const QflashKernelArgs& a) {
    constexpr int kRows = 1024 / D;                 // rows of a 1 KiB piece
    constexpr int kPieces = BC / kRows;             // pieces of K, or V, of a tile
    constexpr int kRowPieces = D / 16;              // 16-byte pieces of a row
    constexpr bool SB = XM == kExpTable;
    if (!QMAX) round_down();
    const int N = a.N;
    const int unit = qflash_unit_of_workgroup(blockIdx.x, a.units_per_xcd, a.xcd_period);
    if (unit >= a.n_units) return;
    const int qt = unit % a.n_qtiles, bh = unit / a.n_qtiles;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_waves = (int)(blockDim.x >> 6);
    const int g = lane >> 5, li = lane & 31;
    const QflashHeadConsts hc = head_consts(a, bh);
    const auto c = make_exp_const<XM != kExpTable || MIXED != 0>(hc);
    // (made anew where the compiler would otherwise hold, or spill, them through a tile)
    auto lane_offsets = [&]() {
        int l = (int)threadIdx.x & 63;
        asm volatile("" : "+v"(l));
        return swizzled_lane_offsets<D>(l);
    };
    SwizzledLane sl = lane_offsets();

    // ---- LDS: [weight table][three or four slots]; the dynamic LDS is the only LDS of the kernel, so the
    //      table index is its address
    const int lds0 = (int)(size_t)(lds_void)smem_ring;
    const int tbytes = XM == kExpTable ? a.ring_table_lds : 0;
    const int ring_base = lds0 + tbytes;

    const size_t head_off = (size_t)bh * N * D;
    const int8_t* Kh = a.K + head_off;
    const int8_t* Vh = a.V + head_off;
    const int row0 = qt * a.rows_per_wg + wave * 32;
    const bool active = row0 < N;
    const int n_tiles = (N + BC - 1) / BC;

    // Lane part of the address of a 1 KiB piece: row lane / (D / 16), 16-byte piece lane % (D / 16) permuted
    // by the row.  Rows beyond the sequence are clamped to the last row (their weights are masked).
    auto lane_row = [](int l) { return l / kRowPieces; };
    auto lane_piece = [&](int l) { return ((l ^ (lane_row(l) >> 2)) & (kRowPieces - 1)) << 4; };
    const int lane_off = lane_row(lane) * D + lane_piece(lane);
    // LDS slots of one tile of K or V each.  With 32 features two of K and two of V; with 64 three that change places:
    // V of tile j + 1 goes where K of tile j was, K of tile j + 2 where V of tile j was.
    constexpr int kSlot = BC * D;
    constexpr bool kThree = qflash_ring_slots(D) == 3;
    int k_slot = ring_base, v_slot = ring_base + kSlot, k_next = ring_base + 2 * kSlot, v_next = kThree ? k_slot : ring_base + 3 * kSlot;
    auto next_slots = [&]() {
        if (kThree) {
            const int free = v_slot;
            v_slot = k_slot;
            k_slot = k_next;
            k_next = free;
            v_next = k_slot;
        } else {
            const int k = k_slot, v = v_slot;
            k_slot = k_next;
            v_slot = v_next;
            k_next = k;
            v_next = v;
        }
    };
    // Requests the 1 KiB pieces of tile j, dealt round robin to the wavefronts: FROM 0 to TO 1: K, 1 to 2: V, 0 to 2: both.
    // EDGE: the tile may reach beyond the sequence, or not exist.
    auto request = [&](int j, int k_lds, int v_lds, auto from, auto to, auto edge) {
        constexpr int X0 = decltype(from)::value * kPieces, X1 = decltype(to)::value * kPieces;
        constexpr bool EDGE = decltype(edge)::value != 0;
        [[maybe_unused]] int l = 0;
        if (EDGE) {
            if (j >= n_tiles) return;
            l = (int)threadIdx.x & 63;
            asm volatile("" : "+v"(l));
        }
        for (int x = X0 + wave; x < X1; x += n_waves) {
            const bool is_k = x < kPieces;
            const int b = is_k ? x : x - kPieces;
            const int8_t* Th = is_k ? Kh : Vh;
            const int lds = (is_k ? k_lds : v_lds) + 1024 * b;
            load_1k_to_lds(Th, EDGE ? min(BC * j + kRows * b + lane_row(l), N - 1) * D + lane_piece(l) : lane_off + kSlot * j + 1024 * b, lds);
        }
    };
    auto request_next = [&](int j, auto from, auto to) {
        if (__builtin_expect(BC * (j + 1) <= N, 1)) request(j, k_next, v_next, from, to, RingInt<0>{});
        else request(j, k_next, v_next, from, to, RingInt<1>{});
    };

    // ---- prologue: table (shared), first tile, this lane's query row (straight to its operand
    //      registers; rows beyond the sequence read the last row and are never stored); one wait,
    //      one barrier.  The query registers are touched right after the wait: these are the only
    //      loads the compiler counts, and it must not find them pending later, when waiting for
    //      them would mean waiting for the tile in flight.
    if (XM == kExpTable)
        for (int it = wave; it < ((hc.lut_bytes + 1023) >> 10); it += n_waves)
            load_1k_to_lds((const int8_t*)hc.lut + 1024 * it, 16 * lane, lds0 + 1024 * it);
    request(0, k_slot, v_slot, RingInt<0>{}, RingInt<2>{}, RingInt<1>{});
    v4i qreg[D / 32];
    {
        const int8_t* Qrow = a.Q + head_off + (size_t)min(row0 + li, N - 1) * D + 16 * g;
#pragma unroll
        for (int s = 0; s < D / 32; ++s) qreg[s] = *(const v4i*)(Qrow + 32 * s);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < D / 32; ++s) asm volatile("" : "+v"(qreg[s]));
    __syncthreads();

    RowState<D> st;
    st.l = 0;
    const int m_init = QMAX ? qmax_initial_reference(hc.s_inv, hc.a_mul) : kMInit;
    st.m = SB ? (int)((unsigned)m_init + (unsigned)kAccBias) : m_init;

    const int n_full = N / BC, rem = N - n_full * BC;
    // The next tile lands while this one is computed.  Four slots: one barrier behind the tile, after every wavefront has
    // waited for its own loads, publishes the next tile and frees the slots of this one.  Three: K of the next tile is
    // requested ahead of this one and V behind it; a barrier between the weights and the first read of V
    // publishes and frees the slot of K, one behind the tile frees that of V.
    auto publish = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    int jt = 0;                                          // the tile
    auto before_v = [&]() {
        if (kThree) publish();
    };
#define QF_RING_COMPUTE(FULL_, FIRST_, NV_, NG_, FR_)                                                              \
    {                                                                                                              \
        int g_ = 0;                                                                                                \
        if (!(FULL_)) {      /* (nothing of it is to be prepared ahead of the tiles) */                            \
            g_ = (int)threadIdx.x & 63;                                                                            \
            asm volatile("; ragged tile %1" : "+v"(g_) : "i"(NG_) : "memory");                                     \
            sl = swizzled_lane_offsets<D>(g_);                                                                     \
            g_ >>= 5;                                                                                              \
        }                                                                                                          \
        process_tile<D, BC, kBiasNone, XM, SB, FULL_, FIRST_, kLaySwizzled, NG_, QMAX, ring_release<QMAX>(FR_), MIXED>( \
            st, qreg, nullptr, 0, nullptr, 0, NV_, hc.lut_xp, nullptr, nullptr, c, hc.a_mul, li, g_,               \
            k_slot + sl.k_off, v_slot + sl.v_off, before_v);                                                       \
    }
#define QF_RING_TILE(FIRST_, FR_)                                                                                  \
    {                                                                                                              \
        request_next(jt + 1, RingInt<0>{}, RingInt<kThree ? 1 : 2>{});                                             \
        if (active) QF_RING_COMPUTE(true, FIRST_, BC, 0, FR_)                                                      \
        else before_v();                                                                                           \
        if (kThree) {                                                                                              \
            request_next(jt + 1, RingInt<1>{}, RingInt<2>{});                                                      \
            __syncthreads();                                                                                       \
        } else {                                                                                                   \
            publish();                                                                                             \
        }                                                                                                          \
        next_slots();                                                                                              \
        ++jt;                                                                                                      \
    }
#define QF_RING_LAST(FIRST_, NG_, FR_) QF_RING_COMPUTE(false, FIRST_, rem, NG_, FR_)
    constexpr bool kFloats = XM == kExpTable && !QMAX;
    // up to this many keys, the last tile takes code for (twice) the groups there are; as many kinds of it as registers allow
    constexpr int kPartial = D == 32 && BC == 128 ? 128 : 16;
    // (N >= BC but for 32 features and tiles of 128)
    if (D == 64 || BC == 64 || n_full > 0) {
        // wavefronts of the last workgroups give way the further they have come (qflash_plan_ring)
        int give_way = (int)blockIdx.x >= a.ring_even_from ? n_tiles / 2 : n_tiles;
        if (a.ring_even_from < (int)gridDim.x) __builtin_amdgcn_s_setprio(3);
        auto priority = [&]() {
            if (__builtin_expect(jt == give_way, 0)) {           // at a half, three quarters and seven eighths of the tiles
                if (give_way == n_tiles / 2) {
                    __builtin_amdgcn_s_setprio(2);
                    give_way = (3 * n_tiles) / 4;
                } else if (give_way == (3 * n_tiles) / 4) {
                    __builtin_amdgcn_s_setprio(1);
                    give_way = (7 * n_tiles) / 8;
                } else {
                    __builtin_amdgcn_s_setprio(0);
                }
            }
        };
        QF_RING_TILE(true, true)
        sl = lane_offsets();
        // (every wavefront passes the barrier of every tile in one of the two loops)
        while (jt < n_full && __builtin_expect(__builtin_amdgcn_ballot_w64(st.l >= kFloatReleaseMaxL) == 0, 1)) {
            priority();
            QF_RING_TILE(false, true)
        }
        while (jt < n_full) {
            priority();
            QF_RING_TILE(false, false)
        }
        if (!active) {
            if (rem > 0) before_v();
            return;
        }
        if (rem == 0) {
        } else if (!kFloats || (rem > kPartial) || __builtin_amdgcn_ballot_w64(st.l >= kFloatReleaseMaxL) != 0) {
            if (kFloats && (D == 32 || BC == 128) && __builtin_amdgcn_ballot_w64(st.l >= kFloatReleaseMaxL) == 0) QF_RING_LAST(false, 0, true)
            else QF_RING_LAST(false, 0, false)
        } else if constexpr (kFloats) {
            const int ng = (rem + 7) >> 3;
            if (ng == 1) QF_RING_LAST(false, -1, true)
            else if constexpr (kPartial >= 16) {
                if (ng == 2) QF_RING_LAST(false, -2, true)
                else if constexpr (kPartial == 128) {
                if (ng <= 4) QF_RING_LAST(false, -4, true)
                else if (ng <= 8) QF_RING_LAST(false, -8, true)
                else QF_RING_LAST(false, -BC / 8, true)
                }
            }
        }
    } else if constexpr (D == 32 && BC == 128) {
        if (!active) return;
        QF_RING_LAST(true, 0, true)
    }
    int lane_ = (int)threadIdx.x & 63;              // (made anew: no register is held for it through the tiles)
    asm volatile("" : "+v"(lane_));
    const int i = row0 + (lane_ & 31);
    if (i < N) normalise_store<D, 20, acc_offset<ring_release<QMAX>(true)>()>(st, a.O + head_off + (size_t)i * D, lane_ >> 5, a.out_round != 0);
#undef QF_RING_LAST
#undef QF_RING_COMPUTE
#undef QF_RING_TILE
}

// Wavefronts per SIMD the register allocation has to allow (a single spilled register costs microseconds: every
// wavefront's scratch goes through memory).  64 features: with KV tiles of 64, 5 for the look-up variant (91 registers)
// and 4 for the others; 4 with tiles of 128 (128 registers; three wavefronts, 137 registers: 384 pairs of 577 tokens
// 36.6 us instead of 33.8, also because an odd number of wavefronts does not share a SIMD evenly: 5.3 cycles per integer
// instruction with three, 4.1 with two or four).  32 features: 5 and 4 (78 and 111 registers).
template <int D, int BC, int XM>
constexpr int ring_min_waves() {
    if (D == 32) return BC == 128 ? 4 : 5;
    return BC == 128 ? 4 : XM == kExpTable ? 5 : 4;
}

// QMAX: the quantised-maximum variant (not Algorithm 1 as printed; see process_tile).
template <int D, int BC, int XM, bool QMAX, int MIXED = 0>
__global__ __launch_bounds__(64 * kRingMaxWaves, (ring_min_waves<D, BC, XM>())) void qflash_fwd_ring(const QflashKernelArgs a) {
    if constexpr (XM == kExpAuto) {
        const int unit = qflash_unit_of_workgroup(blockIdx.x, a.units_per_xcd, a.xcd_period);
        if (unit >= a.n_units) return;
        const int table = head_consts(a, unit / a.n_qtiles).lut_bytes;
        if (D == 32 && table >= kRingMixedBytes) ring_body<D, BC, kExpTable, QMAX, D == 32 ? 2 : 0>(a);
        else if (table > 0) ring_body<D, BC, kExpTable, QMAX>(a);
        else ring_body<D, BC, kExpShift, QMAX>(a);
    } else {
        ring_body<D, BC, XM, QMAX, MIXED>(a);
    }
}

template <int D, int BC, int XM, bool QMAX, int MIXED = 0>
int launch_ring(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    return qflash_launch_kernel<qflash_fwd_ring<D, BC, XM, QMAX, MIXED>>(a, (unsigned)(8 * a.units_per_xcd), (unsigned)(64 * a.waves_per_head), lds, lds_limit, st);
}

}  // namespace

namespace {
template <int D, int BC, bool QMAX>
int launch_mode(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    if (a.exp_mode == kExpAuto) return launch_ring<D, BC, kExpAuto, QMAX>(a, lds, lds_limit, st);
    if (D == 32 && a.exp_mode == kExpTable && a.lut_bytes_max >= kRingMixedBytes) {
        // (at most one workgroup to a compute unit; measured to make no difference where the kernel chooses, kExpAuto)
        if (a.n_units <= (a.n_cu > 0 ? a.n_cu : 256)) return launch_ring<D, BC, kExpTable, QMAX, D == 32 ? 1 : 0>(a, lds, lds_limit, st);
        return launch_ring<D, BC, kExpTable, QMAX, D == 32 ? 2 : 0>(a, lds, lds_limit, st);
    }
    if (a.exp_mode == kExpTable) return launch_ring<D, BC, kExpTable, QMAX>(a, lds, lds_limit, st);
    if (a.exp_mode == kExpShift0) return launch_ring<D, BC, kExpShift0, QMAX>(a, lds, lds_limit, st);
    return launch_ring<D, BC, kExpShift, QMAX>(a, lds, lds_limit, st);
}
template <bool QMAX>
int launch_variant(const QflashKernelArgs& a, int d, size_t lds, int lds_limit, hipStream_t st) {
    if (d == 64) return a.kv_tile == 64 ? launch_mode<64, 64, QMAX>(a, lds, lds_limit, st) : launch_mode<64, 128, QMAX>(a, lds, lds_limit, st);
    return a.kv_tile == 64 ? launch_mode<32, 64, QMAX>(a, lds, lds_limit, st) : launch_mode<32, 128, QMAX>(a, lds, lds_limit, st);
}
}  // namespace

int qflash_launch_fwd_ring(const QflashKernelArgs& a, int d, int lds_limit, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    // everything the kernel's indexing assumes, checked once more where it is launched
    if (!a.ring_dma || !a.ring || a.bias || a.heads_per_wg != 1 || (a.kv_tile != 64 && a.kv_tile != 128) || (d != 32 && d != 64))
        return (int)hipErrorInvalidValue;
    if (a.waves_per_head < 1 || a.waves_per_head > kRingMaxWaves || a.rows_per_wg != 32 * a.waves_per_head) return (int)hipErrorInvalidValue;
    if ((long long)a.rows_per_wg * a.n_qtiles < a.N) return (int)hipErrorInvalidValue;
    if (a.N < a.kv_tile && (d == 64 || a.kv_tile == 64)) return (int)hipErrorInvalidValue;
    const bool table = a.exp_mode == kExpTable || a.exp_mode == kExpAuto;
    if (table && a.lut_bytes_max > a.ring_table_lds) return (int)hipErrorInvalidValue;
    const size_t lds = qflash_ring_lds_bytes(a.waves_per_head, a.kv_tile, table ? a.ring_table_lds : 0, d);
    if (lds > (size_t)lds_limit) return (int)hipErrorInvalidValue;
    return a.qmax ? launch_variant<true>(a, d, lds, lds_limit, st) : launch_variant<false>(a, d, lds, lds_limit, st);
}
