// gfx950 kernel of the integer-only fused attention forward pass (Algorithm 1) for long sequences
// without a bias: the two-tile ring, fed by direct global-to-LDS loads.
//
// A workgroup of up to 8 wavefronts serves 32 query rows per wavefront of one (batch, head) pair and
// walks over all KV tiles of the pair.  LDS holds the weight table and two KV tiles: the one in use
// and the one on its way.  K and V tiles arrive row-major as they lie in memory (16-byte pieces
// permuted by the row so that operand reads are free of bank conflicts), put there by `global_load_lds_dwordx4`; the K/Q operands are plain 16-byte LDS reads
// and the V^T operand is read with the transposing 8-bit LDS read (see qflash_tile.h).  Compared with
// staging through registers (qflash_resident.h) there are no staging registers, no byte transposes
// in the vector ALU and no LDS write instructions: about a third of that kernel's vector
// instructions on these shapes.
//
// What bounds it, by counters (cycles of a compute unit at 2.2 GHz per wavefront and KV tile: a vector instruction 4 on
// one of four SIMDs, an LDS operand read 8 or, transposing, 4, a look-up 2.5 plus the counted bank conflicts):
//   64 features, tiny table (256 pairs of 577 tokens, tiles of 64, 26 us): 302 measured; 214 vector, 63 matrix, 130
//     LDS, no bank conflicts.  No unit is full.  The vector and the matrix time add up: the barrier after every
//     tile keeps the wavefronts of a workgroup in one phase.
//   64 features, tiles of 128 (384 pairs of 577, 39 us): 604 measured; 338 vector, 125 matrix, 350 LDS (1.5 conflict
//     cycles per look-up).  No unit is full here either: 137 registers leave three wavefronts to a SIMD.
//   32 features (64 pairs of 2100 tokens, 73 us): 295 measured; 191 vector, 33 matrix, 251 LDS, 219 of them 28 look-ups
//     with 5.3 conflict cycles each: here the look-ups are most of the time.
// 32 features against the streamed kernel that staged one tile at a time through registers and computed the
// weights: B*H = 64, N = 2100 145.6 -> 73 us with tiles of 64, 202 -> 77.5 us with tiles of 128; against whole
// sequences in LDS: B*H = 96, N = 1200 56.8 -> 39.6 us.
//
// Synchronisation: the wavefronts share the loads of a tile (1 KiB pieces, dealt round robin).
// While tile j is computed, tile j+1 lands in the other slot; after its arithmetic a wavefront waits
// for its own loads (vmcnt) and then for the others at a workgroup barrier, which also says that
// everybody is done with tile j, whose slot the loads of tile j+2 may now overwrite.  Every
// wavefront of a workgroup executes every barrier, with or without query rows of its own.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "qflash_launch.h"
#include "qflash_tile.h"

// (M0 is written by the direct loads below and declared as clobbered)
#pragma clang diagnostic ignored "-Winline-asm"

namespace {

extern __shared__ __align__(1024) int8_t smem_ring[];

// Weight tables of 32 features from this size on: part of the weights is computed (MIXED of process_tile).
constexpr int kRingMixedBytes = 7 * 1024;

template <int D, int BC, int XM, bool QMAX, bool MIXED = false>
__device__ __forceinline__ void ring_body(const QflashKernelArgs& a) {
    constexpr int kRingTileBytes = 2 * BC * D;      // one KV tile in LDS: K (BC rows of D bytes), then V
    constexpr int kRows = 1024 / D;                 // rows of a 1 KiB piece
    constexpr int kPieces = 2 * BC / kRows;         // pieces of a tile: K, then V
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
    const ExpConst c = make_exp_const<XM != kExpTable || MIXED>(hc);
    const SwizzledLane sl = swizzled_lane_offsets<D>(lane);

    // ---- LDS: [weight table][slot 0][slot 1]; the dynamic LDS is the only LDS of the kernel, so the
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
    // The 1 KiB pieces of tile j (the K blocks, then the V blocks), dealt round robin to the wavefronts.
    auto issue_tile = [&](int j) {
        const int slot = ring_base + kRingTileBytes * (j & 1);
        if (BC * (j + 1) <= N) {
            for (int x = wave; x < kPieces; x += n_waves)
                load_1k_to_lds(x < kPieces / 2 ? Kh : Vh, lane_off + BC * D * j + 1024 * (x % (kPieces / 2)), slot + 1024 * x);
        } else {
            int l = (int)threadIdx.x & 63;
            asm volatile("" : "+v"(l));
            for (int x = wave; x < kPieces; x += n_waves)
                load_1k_to_lds(x < kPieces / 2 ? Kh : Vh, min(BC * j + kRows * (x % (kPieces / 2)) + lane_row(l), N - 1) * D + lane_piece(l), slot + 1024 * x);
        }
    };

    // ---- prologue: table (shared), first tile, this lane's query row (straight to its operand
    //      registers; rows beyond the sequence read the last row and are never stored); one wait,
    //      one barrier.  The query registers are touched right after the wait: these are the only
    //      loads the compiler counts, and it must not find them pending later, when waiting for
    //      them would mean waiting for the tile in flight.
    if (XM == kExpTable)
        for (int it = wave; it < ((hc.lut_bytes + 1023) >> 10); it += n_waves)
            load_1k_to_lds((const int8_t*)hc.lut + 1024 * it, 16 * lane, lds0 + 1024 * it);
    issue_tile(0);
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
#define QF_RING_COMPUTE(FULL_, FIRST_, J_, NV_, NG_, FR_)                                                          \
    {                                                                                                              \
        const int slot = ring_base + kRingTileBytes * ((J_) & 1);                                                  \
        int k_off = sl.k_off, v_off = sl.v_off, g_ = 0;                                                            \
        if (!(FULL_)) {      /* (nothing of it is to be prepared ahead of the tiles) */                            \
            g_ = (int)threadIdx.x & 63;                                                                            \
            asm volatile("; ragged tile %3" : "+v"(g_), "+v"(k_off), "+v"(v_off) : "i"(NG_) : "memory");           \
            g_ >>= 5;                                                                                              \
        }                                                                                                          \
        process_tile<D, BC, kBiasNone, XM, SB, FULL_, FIRST_, kLaySwizzled, NG_, QMAX, FR_, MIXED>(                \
            st, qreg, nullptr, 0, nullptr, 0, NV_, hc.lut_xp, nullptr, nullptr, c, hc.a_mul, li, g_,               \
            slot + k_off, slot + BC * D + v_off);                                                                  \
    }
#define QF_RING_TILE(FIRST_, J_, FR_)                                                                              \
    {                                                                                                              \
        if ((J_) + 1 < n_tiles) issue_tile((J_) + 1);                                                              \
        if (active) QF_RING_COMPUTE(true, FIRST_, J_, BC, 0, FR_)                                                  \
        if ((J_) + 1 < n_tiles) {                                                                                  \
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                                                       \
            __syncthreads();                                                                                       \
        }                                                                                                          \
    }
#define QF_RING_LAST(FIRST_, J_, NV_, NG_, FR_) { QF_RING_COMPUTE(false, FIRST_, J_, NV_, NG_, FR_) }
    constexpr bool kFloats = XM == kExpTable && !QMAX;
    // (N >= BC but for 32 features and tiles of 128)
    if (D == 64 || BC == 64 || n_full > 0) {
        // wavefronts of the last workgroups give way the further they have come (qflash_plan_ring)
        const bool even = (int)blockIdx.x >= a.ring_even_from;
        const int p2 = even ? n_tiles / 2 : n_tiles, p1 = even ? (3 * n_tiles) / 4 : n_tiles, p0 = even ? (7 * n_tiles) / 8 : n_tiles;
        if (a.ring_even_from < (int)gridDim.x) __builtin_amdgcn_s_setprio(3);
        QF_RING_TILE(true, 0, true)
        int j = 1;
        // (every wavefront passes the barrier of every tile in one of the two loops)
        for (; j < n_full && __builtin_amdgcn_ballot_w64(st.l >= kFloatReleaseMaxL) == 0; ++j) {
            if (j == p2) __builtin_amdgcn_s_setprio(2);
            if (j == p1) __builtin_amdgcn_s_setprio(1);
            if (j == p0) __builtin_amdgcn_s_setprio(0);
            QF_RING_TILE(false, j, true)
        }
        for (; j < n_full; ++j) QF_RING_TILE(false, j, false)
        if (!active) return;
        if (rem == 0) {
        } else if (!kFloats || (BC == 64 && rem > 16) || __builtin_amdgcn_ballot_w64(st.l >= kFloatReleaseMaxL) != 0) {
            if (kFloats && D == 32 && __builtin_amdgcn_ballot_w64(st.l >= kFloatReleaseMaxL) == 0) QF_RING_LAST(false, n_full, rem, 0, true)
            else QF_RING_LAST(false, n_full, rem, 0, false)
        } else if constexpr (kFloats) {
            const int ng = (rem + 7) >> 3;
            if (ng == 1) QF_RING_LAST(false, n_full, rem, -1, true)
            else if (ng == 2) QF_RING_LAST(false, n_full, rem, -2, true)
            else if constexpr (BC == 128) {
                if (ng <= 4) QF_RING_LAST(false, n_full, rem, -4, true)
                else if (ng <= 8) QF_RING_LAST(false, n_full, rem, -8, true)
                else QF_RING_LAST(false, n_full, rem, -BC / 8, true)
            }
        }
    } else if constexpr (D == 32 && BC == 128) {
        if (!active) return;
        QF_RING_LAST(true, 0, rem, 0, true)
    }
    const int i = row0 + li;
    if (i < N) normalise_store<D, 20, acc_offset<QMAX>()>(st, a.O + head_off + (size_t)i * D, g, a.out_round != 0);
#undef QF_RING_LAST
#undef QF_RING_COMPUTE
#undef QF_RING_TILE
}

// Wavefronts per SIMD the register allocation has to allow.  64 features: with KV tiles of 64, 5 for the
// look-up variant (94 registers) and 4 for the others (which would spill at 96); 3 with tiles of 128 (137
// registers; held to 128 it spills a dozen and is a sixth slower).  32 features: 5 and 4 (72 and 104
// registers).
template <int D, int BC, int XM>
constexpr int ring_min_waves() {
    if (D == 32) return BC == 128 ? 4 : 5;
    return BC == 128 ? 3 : XM == kExpTable ? 5 : 4;
}

// QMAX: the quantised-maximum variant (not Algorithm 1 as printed; see process_tile).
template <int D, int BC, int XM, bool QMAX, bool MIXED = false>
__global__ __launch_bounds__(64 * kRingMaxWaves, (ring_min_waves<D, BC, XM>())) void qflash_fwd_ring(const QflashKernelArgs a) {
    if constexpr (XM == kExpAuto) {
        const int unit = qflash_unit_of_workgroup(blockIdx.x, a.units_per_xcd, a.xcd_period);
        if (unit >= a.n_units) return;
        const int table = head_consts(a, unit / a.n_qtiles).lut_bytes;
        if (D == 32 && table >= kRingMixedBytes) ring_body<D, BC, kExpTable, QMAX, D == 32>(a);
        else if (table > 0) ring_body<D, BC, kExpTable, QMAX>(a);
        else ring_body<D, BC, kExpShift, QMAX>(a);
    } else {
        ring_body<D, BC, XM, QMAX, MIXED>(a);
    }
}

template <int D, int BC, int XM, bool QMAX, bool MIXED = false>
int launch_ring(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    return qflash_launch_kernel<qflash_fwd_ring<D, BC, XM, QMAX, MIXED>>(a, (unsigned)(8 * a.units_per_xcd), (unsigned)(64 * a.waves_per_head), lds, lds_limit, st);
}

}  // namespace

namespace {
template <int D, int BC, bool QMAX>
int launch_mode(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    if (a.exp_mode == kExpAuto) return launch_ring<D, BC, kExpAuto, QMAX>(a, lds, lds_limit, st);
    if (D == 32 && a.exp_mode == kExpTable && a.lut_bytes_max >= kRingMixedBytes) return launch_ring<D, BC, kExpTable, QMAX, D == 32>(a, lds, lds_limit, st);
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
