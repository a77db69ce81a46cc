// Host-only part of the library: everything that decides about a call without touching the GPU --
// derivation of the integer constants from the real scales, the argument checks of the attention
// entry points, and the choice of kernel and work decomposition.  Plain C++ (no HIP): this file is
// also compiled, together with the CPU oracle, into a sanitizer build (address + undefined
// behaviour) that the tests without a GPU run.
#include <cmath>
#include <cstddef>
#include <cstdint>

#include "qflash.h"
#include "qflash_internal.h"
#include "qflash_derive.h"

extern "C" int qflash_params_from_scales(double sQ, double sK, double sV, int d, qflash_params* out) {
    if (!out) return QFLASH_ERR_NULL;
    if (d != 32 && d != 64) return QFLASH_ERR_SHAPE;
    if (!(sQ > 0.0) || !(sK > 0.0) || !(sV > 0.0) || !std::isfinite(sQ) || !std::isfinite(sK) ||
        !std::isfinite(sV))
        return QFLASH_ERR_PARAM;
    return qflash_derive_params(sQ, sK, std::sqrt((double)d), out);
}

// The argument checks shared by every attention entry point, in the order the header documents.
// consts_on_device: the integer constants are computed on the GPU (dynamic quantisation), p is unused.
int qflash_check_call(const void* Q, const void* K, const void* V, const void* O, const int32_t* bias, int bias_B,
                      int bias_H, bool bias_packed, int B, int H, int N, int d, int kv_tile, const qflash_params* p,
                      bool per_head, bool consts_on_device, bool qmax) {
    if (!Q || !K || !V || !O || (!p && !consts_on_device)) return QFLASH_ERR_NULL;
    if (d != 32 && d != 64) return QFLASH_ERR_SHAPE;
    if (B < 1 || H < 1 || N < 1 || N > QFLASH_MAX_N) return QFLASH_ERR_SHAPE;
    if ((int64_t)B * H * N * d >= ((int64_t)1 << 31)) return QFLASH_ERR_SHAPE;
    if (per_head && H > QFLASH_MAX_PARAM_HEADS) return QFLASH_ERR_SHAPE;
    if (bias) {
        if (bias_B < 1 || bias_H < 1) return QFLASH_ERR_SHAPE;
        if ((int64_t)bias_B * bias_H * N * N >= ((int64_t)1 << 31)) return QFLASH_ERR_SHAPE;
        if (bias_packed && qflash_packed_bias_words(bias_B * bias_H, N) >= ((int64_t)1 << 29)) return QFLASH_ERR_SHAPE;
    } else if (bias_packed) {
        return QFLASH_ERR_NULL;
    }
    if (kv_tile != 64 && kv_tile != 128) return QFLASH_ERR_TILE;
    const int n_p = consts_on_device ? 0 : per_head ? H : 1;
    for (int h = 0; h < n_p; ++h) {
        if (!qflash_params_ok(p[h])) return QFLASH_ERR_PARAM;
        if (p[h].out_round != p[0].out_round) return QFLASH_ERR_PARAM;   // one rounding mode per call
        if (qmax && p[h].x_shift != 0) return QFLASH_ERR_PARAM;
    }
    if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)O) & 15u) return QFLASH_ERR_ALIGN;
    if (bias && ((uintptr_t)bias & (bias_packed ? 15u : 3u))) return QFLASH_ERR_ALIGN;
    return QFLASH_OK;
}

long long qflash_packed_bias_words(int slices, int N) {
    const long long nb = (N + 31) / 32;
    return (long long)slices * nb * nb * 256;
}

// Table size assumed when deciding whether two workgroups with the whole sequence in LDS fit a compute unit.
constexpr int kRingTableGuess = 32 * 1024;

// LDS bytes of the resident kernel: K and V^T of `heads` heads of N rows (ring: of two KV tiles)
// and the weight table; 0 if they do not fit.
size_t qflash_resident_lds_bytes(int N, int d, int heads, int table_bytes, int lds_limit, int ring_tile) {
    const size_t npad = (size_t)((N + 31) & ~31);
    const size_t kv = ring_tile ? 2 * ((size_t)ring_tile * (size_t)(d + 16) + (size_t)d * (size_t)(ring_tile + 16))
                                : npad * (size_t)(d + 16) + (size_t)d * (npad + 16);
    const size_t bytes = (size_t)heads * kv + (size_t)table_bytes;
    return bytes <= (size_t)lds_limit ? bytes : 0;
}

int qflash_plan_fwd(int BH, int N, int d, int kv_tile, int lds_limit, QflashKernelArgs* a) {
    a->resident = qflash_resident_lds_bytes(N, d, 1, 0, lds_limit) != 0;
    a->heads_per_wg = 1;
    a->pipelined = 0;
    a->ring = 0;
    a->ring_dma = 0;
    a->kv_tile = kv_tile;
    // Long sequences: K and V^T of the whole sequence (plus a weight table) would leave room for
    // one workgroup per compute unit, or for none.  Where the kernel variant can stage tile by
    // tile (d = 64, tile 64), LDS holds two tiles only and workgroups are at most 8 wavefronts,
    // so that two of them share a compute unit.
    const bool two_fit = qflash_resident_lds_bytes(N, d, 1, kRingTableGuess, lds_limit / 2) != 0;
    // (without a bias the ring fed by direct loads is the faster kernel for every long sequence)
    if (d == 64 && N > 256 && (kv_tile == 128 || !two_fit || !a->bias)) {
        const int nblk = (N + 31) / 32;
        const int cus = a->n_cu > 0 ? a->n_cu : 256;
        int waves;
        // Without a bias the ring is fed by direct global-to-LDS loads (qflash_fwd_ring): no wavefront
        // stages anything, and workgroups of four wavefronts, one per SIMD, are where qflash_plan_ring starts from.
        a->ring_dma = !a->bias ? 1 : 0;
        if (a->ring_dma) {
            const int tiles = (nblk + 3) / 4;
            waves = (nblk + tiles - 1) / tiles;                   // balanced: at most 4
        } else if (kv_tile == 128) {
            // 160-odd registers leave three wavefront slots per SIMD: three workgroups of four
            // wavefronts (which is also what stages a tile: 256 threads, two items each)
            waves = 4;
        } else {
            // Workgroups of up to 8 wavefronts (two per compute unit: 128 registers leave four
            // wavefront slots per SIMD) or of 4 (four per compute unit, one wavefront on every SIMD,
            // but every wavefront then also stages K/V): whichever gives the busiest compute unit
            // fewer workgroups to run one after the other.
            const int tiles8 = (nblk + 7) / 8, tiles4 = (nblk + 3) / 4;
            const long long turns8 = ((long long)BH * tiles8 + 2ll * cus - 1) / (2ll * cus);
            const long long turns4 = ((long long)BH * tiles4 + 4ll * cus - 1) / (4ll * cus);
            int tiles = turns4 < turns8 ? tiles4 : tiles8;
            if ((nblk + tiles - 1) / tiles < 4) tiles = tiles8;   // staging needs 256 threads
            waves = (nblk + tiles - 1) / tiles;                   // balanced: 4..8
        }
        a->resident = 1;
        a->ring = 1;
        a->pipelined = 1;
        a->rows_per_wg = 32 * waves;
        a->waves_per_head = waves;
    } else if (a->resident) {
        const int nblk = (N + 31) / 32;
        const int max_waves = N <= 256 ? kResidentMaxWavesNarrow : kResidentMaxWavesWide;
        const int tiles = (nblk + max_waves - 1) / max_waves;
        const int waves = (nblk + tiles - 1) / tiles;       // balanced
        a->rows_per_wg = 32 * waves;
        a->waves_per_head = waves;
        // Short sequences (windowed attention): several (batch, head) pairs per workgroup, so that
        // a workgroup is 8 wavefronts and a weight table is staged once for all of them.
        if (tiles == 1 && waves <= 4) {
            int hp = kResidentMaxWavesNarrow / waves;
            if (hp > BH) hp = BH;
            while (hp > 1 && qflash_resident_lds_bytes(N, d, hp, 0, lds_limit / 4) == 0) --hp;
            a->heads_per_wg = hp;
        }
        // Tile-by-tile staging needs a second KV tile to overlap with and 256 staging threads
        // (32-byte pieces of K plus 4x8 blocks of V of one tile, one or two items per thread).
        a->pipelined = a->heads_per_wg == 1 && N > kv_tile && waves >= 4;
    } else {
        a->rows_per_wg = kStreamRows;
        a->waves_per_head = kStreamWaves;
    }
    a->n_qtiles = (N + a->rows_per_wg - 1) / a->rows_per_wg;
    // per-head constants with several pairs per workgroup: group by head (see the kernel)
    a->same_head = a->per_head && a->heads_per_wg > 1 ? 1 : 0;
    const long long units = a->same_head ? (long long)((a->B + a->heads_per_wg - 1) / a->heads_per_wg) * a->H
                            : a->heads_per_wg > 1 ? ((long long)BH + a->heads_per_wg - 1) / a->heads_per_wg
                                                  : (long long)BH * a->n_qtiles;
    if (units >= (1ll << 30)) return -1;
    a->n_units = (int)units;
    a->units_per_xcd = (a->n_units + 7) / 8;
    // Bias slices repeat every bias_B * H pairs: see qflash_unit_of_workgroup.
    a->xcd_period = 0;
    if (a->bias) {
        const long long pairs = (long long)a->bias_B * a->H;
        const long long period = a->same_head ? (a->bias_B % a->heads_per_wg == 0 ? pairs / a->heads_per_wg : 0)
                                 : a->heads_per_wg > 1 ? (pairs % a->heads_per_wg == 0 ? pairs / a->heads_per_wg : 0)
                                                       : pairs * a->n_qtiles;
        if (period >= 8 && period % 8 == 0 && period <= units) {
            a->xcd_period = (int)period;
            a->units_per_xcd = (int)(((units + period - 1) / period) * (period / 8));
        }
    }
    return 0;
}

int qflash_table_fits(const QflashKernelArgs& a, int d, int table_bytes, int lds_limit) {
    // Every workgroup copies the table from L2 into its LDS: worth it only while that stays below
    // the bytes of Q, K, V, O the workgroup moves anyway.
    const long long io = 4ll * a.heads_per_wg * a.N * d;
    if (io < (long long)table_bytes) return 0;
    if (a.ring_dma) return qflash_ring_lds_bytes(a.waves_per_head, a.kv_tile, table_bytes, d) <= (size_t)lds_limit / 2;
    // Short sequences with the wide tile: that variant is out of registers with the table's
    // addressing on top (ViT-B/16 B=64: 34 us with the table, 25.5 us without).
    if (d == 64 && a.kv_tile == 128 && a.N <= 256) return 0;
    // keep two workgroups per CU when the sequence is short enough for that to matter
    const int budget = (a.ring || a.N <= 256) ? lds_limit / 2 : lds_limit;
    return qflash_resident_lds_bytes(a.N, d, a.heads_per_wg, table_bytes, budget, a.ring ? a.kv_tile : 0) != 0;
}

size_t qflash_cu_lds_bytes(int N, int heads, int table_bytes) {
    const size_t rows16 = (size_t)((N + 15) & ~15);
    const size_t table = ((size_t)table_bytes + 1023) & ~(size_t)1023;
    return table + (size_t)heads * 3 * rows16 * 64 + 1024 + 4 * (5 * (size_t)heads + 1)
#ifdef QF_TRACE
           + 8 + 2048
#endif
        ;
}

static int plan_cu(int BH, int N, int d, int kv_tile, int lds_limit, int table_bytes, QflashKernelArgs* a, int rounds = 1) {
    a->cu_mode = 0;
    if (d != 64 || a->bias || a->per_head || N > 256) return 0;
    const int cus = a->n_cu > 0 ? a->n_cu : 256;
    const int hpw = (int)(((long long)BH + (long long)cus * rounds - 1) / ((long long)cus * rounds));     // every pair in one round of workgroups (or so many)
    if (qflash_cu_lds_bytes(N, hpw, table_bytes) > (size_t)lds_limit) return 0;
    const int nblk = (N + 31) / 32;
    const int units = hpw * nblk;
    a->cu_mode = 1;
    a->cu_heads = hpw;
    a->cu_groups = (BH + hpw - 1) / hpw;
    const int most = qflash_cu_max_waves(kv_tile);
    a->cu_waves = units < most ? units : most;
    a->cu_table_lds = (table_bytes + 1023) & ~1023;
    return 1;
}

void qflash_cu_reciprocals(QflashKernelArgs* a) {
    a->cu_inv_nblk = qflash_small_reciprocal((unsigned)((a->N + 31) / 32));
    a->cu_inv_per = (unsigned)(0x100000000ull / (unsigned)(3 * ((a->N + 15) / 16))) + 1u;
    a->cu_inv_pairs = qflash_reciprocal((unsigned)a->B * (unsigned)a->H);
    a->cu_inv_b = qflash_reciprocal((unsigned)a->B);
}

int qflash_plan_cu(int BH, int N, int d, int kv_tile, int lds_limit, int table_bytes, QflashKernelArgs* a) {
    a->cu_mode = 0;
    return kv_tile == 64 ? plan_cu(BH, N, d, kv_tile, lds_limit, table_bytes, a) : 0;
}

int qflash_plan_cu128(int BH, int N, int d, int lds_limit, int table_bytes, QflashKernelArgs* a) {
    return plan_cu(BH, N, d, 128, lds_limit, table_bytes, a);
}

int qflash_plan_cu_heads(int BH, int N, int d, int kv_tile, int lds_limit, QflashKernelArgs* a) {
    QflashKernelArgs one = *a;
    one.per_head = 0;
    a->cu_mode = 0;
    if (!a->per_head || N <= 64 || !plan_cu(BH, N, d, kv_tile, lds_limit, 0, &one)) return 0;
    // (with one pair per compute unit, or one KV tile, the resident kernel is as fast: 10.6 us for 192 pairs of
    // 197 tokens against 10.9, 7.8 for 768 pairs of 64 against 8.1; 768 pairs of 197: 24.4 against 22.7)
    if (one.cu_heads < 2) return 0;
    // (two short pairs per compute unit likewise: 360 pairs of 80 tokens 7.1 against 7.7; 516, three per unit, 10.4 against 9.9.
    // With twelve wavefronts, i.e. tiles of 128, it has to fill the chip: 480 pairs of 256 tokens, 240 workgroups,
    // 19.7 against 18.5, but 416 of 197, 208 workgroups, 16.8 against 18.1.)
    const int cus = a->n_cu > 0 ? a->n_cu : 256;
    if (kv_tile == 64 ? one.cu_heads == 2 && N <= 128 : 10 * one.cu_groups < 9 * cus) return 0;
    a->cu_mode = 1;
    a->cu_heads = one.cu_heads;
    a->cu_groups = one.cu_groups;
    a->cu_waves = one.cu_waves;
    const int left = lds_limit - (int)qflash_cu_lds_bytes(N, one.cu_heads, 0);
    a->cu_table_lds = left < kTableMaxBytes ? left & ~1023 : kTableMaxBytes;
    return 1;
}

int qflash_plan_cu_dynamic(int BH, int N, int d, int kv_tile, int lds_limit, QflashKernelArgs* a) {
    // Several rounds of workgroups, as few as hold the pairs, where they do not fit one: a workgroup saves its pairs'
    // int8 copies (write and read) and a kernel whatever its round.  Quantising ahead of the resident kernel -> here, us:
    // 2400 pairs of 197 tokens 216.5 -> 166.7, 1024 of 256 104.6 -> 85.1, 3120 of 100 125.1 -> 88.9, 5440 of 50
    // 103.3 -> 75.9; tiles of 128 likewise.  (int8 tensors: the resident kernel is as fast, no rounds there.)
    const int cus = a->n_cu > 0 ? a->n_cu : 256;
    for (int rounds = 1; rounds <= (BH + cus - 1) / cus; ++rounds) {
        if (!plan_cu(BH, N, d, kv_tile, lds_limit - kCuDynExtraLds, 0, a, rounds)) continue;
        const int left = lds_limit - (int)qflash_cu_lds_bytes(N, a->cu_heads, 0) - kCuDynExtraLds;
        a->cu_table_lds = left < kTableMaxBytes ? left & ~1023 : kTableMaxBytes;
        return 1;
    }
    return 0;
}

// LDS bytes of the direct-load ring kernel: table (rounded up to 1 KiB) and the slots, each of one tile of K or V.
size_t qflash_ring_lds_bytes(int waves, int kv_tile, int table_bytes, int d) {
    (void)waves;
    return (((size_t)table_bytes + 1023) & ~(size_t)1023) + (size_t)qflash_ring_slots(d) * (size_t)kv_tile * (size_t)d;
}

// LDS a workgroup takes on a compute unit of gfx950, which hands it out in pieces of 1280 bytes.  Five workgroups of 32 KiB are
// 160 KiB, all there is, but only four of them are resident; planned as five, with the wrong workgroups giving way, 96 pairs of
// 1200 tokens with 32 features and tiles of 128 took 44.0 us, 32.1 now, 64 of 2100 73.5 and 65.1, 384 of 577 with 64 features
// and tiles of 64 46.3 and 42.1.
static size_t qflash_lds_allocated(size_t bytes) { return (bytes + 1279) / 1280 * 1280; }

// Wavefronts per workgroup of the ring.  More of them share one weight table and one staged tile, fewer
// are dealt out more evenly.  Cost of a choice: wavefronts on the busiest compute unit times the time each
// of them adds, (2200 + 230 x) / x cycles per KV tile with x wavefronts on the unit (fitted to 12 to
// 20: DeiT-B/384, N(0,1), 12 resident: 414; N(0,1.5^2), small table, 20 resident: 341), x limited by LDS and
// registers.  Measured against the fixed four (us): d = 64, 96 pairs of 1025 tokens 47.4 -> 39.7 (seven),
// 36 pairs of 1000 25.2 -> 21.7, 56 of 577 16.7 -> 14.6 (three), 32 features, 96 pairs of 1200 tokens 41.2 -> 39.9 (three).
static double ring_cost(int d, int lds_limit, int table_bytes, const QflashKernelArgs& a, int want, int* waves, int* qtiles, int* resident) {
    const int nblk = (a.N + 31) / 32, cus = a.n_cu > 0 ? a.n_cu : 256;
    *qtiles = (nblk + want - 1) / want;
    const int w = *waves = (nblk + *qtiles - 1) / *qtiles;                        // balanced
    *resident = 1;
    // (at 64 features the SIMDs are busy enough for an uneven workgroup to cost part of its fullest SIMD's share)
    const double eff = d == 64 ? 0.5 * (w + ((w + 3) & ~3)) : w;
    const int per_simd = d == 64 ? (a.kv_tile == 64 ? 5 : 4) : a.kv_tile == 64 ? 6 : 4;   // by registers
    const long long units = (long long)a.B * a.H * *qtiles, per_cu = (units + cus - 1) / cus;
    long long fit = (long long)((size_t)lds_limit / qflash_lds_allocated(qflash_ring_lds_bytes(w, a.kv_tile, table_bytes, d)));
    // Workgroups of five to seven wavefronts do not share the SIMDs evenly, and wait for one another twice a tile.  Tiles of 64: five
    // and six only alone on their compute unit (60 pairs of 513 tokens 14.2 us with six, 15.1 with four; but 384 of 380 26.9 and
    // 21.5, 360 of 330 24.7 and 20.5, 600 of 300 26.5 with five and 23.3); seven and eight even out the rounds (120 of 770 28.3 with
    // seven, 33.3 with four).  Tiles of 128: 384 pairs of 577 47.2 with five and 40.6 with seven, 38.8 with four, 192 of 640 27.6
    // with seven and 22.6; six, and seven in one round, are better all the same where LDS holds two workgroups only, tables of
    // 30 KiB and more (96 of 1025 34.5 with seven, 46.8 with four, 96 of 800 28.4 and 35.4, 240 of 400 16.7 and 22.4, 360 of 330
    // 21.5 with six and 25.0; five 480 of 257 25.6 and 22.4), unless some heads compute their weights (per head, 192 of 350 19.9
    // with six, 16.7 with four, nor three then: 18.3, 288 of 300 24.7 and 20.4).  Three only where the launch does not share out its
    // keys, qflash_plan_split.
    if (d == 64 && a.kv_tile == 64 && (w == 5 || w == 6) && per_cu > 1) return 1e30;
    if (d == 64 && a.kv_tile == 128 && (w == 5 || ((w == 6 || w == 7) && (fit > 2 || a.per_head)) || (w == 7 && per_cu > fit))) return 1e30;
    // 32 features, tiles of 64: six where a compute unit gets three at most (96 of 1025 with a table of 33 KiB 33.1 us with six, 34.9
    // with four; 144 of 1300 65.9 and 51.5, 288 of 530 28.2 and 25.3).  Tiles of 128: six never (240 of 350 12.3 and 11.6, 144 of 1300
    // with a table of 26 KiB 74.6 and 60.7), five where it gets two (160 of 400 11.1 with five, 12.1 with four; 256 of 400 18.3 and
    // 13.9, 128 of 790 29.5 and 22.6, 320 of 410 with a table of 26 KiB 25.0 and 19.2).
    if (d == 32 && a.kv_tile == 64 && w == 6 && per_cu > 3) return 1e30;
    if (d == 32 && a.kv_tile == 128 && (w == 6 || (w == 5 && per_cu > 2))) return 1e30;
    if (d == 64 && want == 3 && ((long long)a.B * a.H * nblk <= 2ll * cus || (a.kv_tile == 128 && a.per_head))) return 1e30;
    const int by_registers = d == 64 && a.kv_tile == 128 ? per_simd / ((w + 3) / 4) : 4 * per_simd / w;
    if (fit > by_registers) fit = by_registers;
    if (fit > per_cu) fit = per_cu;
    if (fit < 1) return 1e30;
    *resident = (int)fit;
    const double x = (double)fit * eff;
    return (double)per_cu * eff * (2200.0 + 230.0 * x) / x;
}

int qflash_plan_ring(int d, int lds_limit, int table_bytes, QflashKernelArgs* a) {
    if (a->bias || a->win_mode || (!a->ring_dma && (d != 32 || a->N <= 64))) return 0;
    const int wants[2][3] = {{4, 8, 3}, {4, 3, 6}};
    double best = 0.0;
    int waves = 0, qtiles = 0, resident = 0;
    for (int i = 0; i < 3; ++i) {
        int w, t, r;
        const double cost = ring_cost(d, lds_limit, table_bytes, *a, wants[d == 32][i], &w, &t, &r);
        if (waves == 0 || cost < 0.97 * best) { best = cost; waves = w; qtiles = t; resident = r; }
    }
    const long long units = (long long)a->B * a->H * qtiles;
    if (units >= (1ll << 30)) return 0;
    a->waves_per_head = waves;
    a->rows_per_wg = 32 * waves;
    a->n_qtiles = qtiles;
    if (d == 32) a->resident = 0;          // (whatever the plan was before: K and V are streamed now)
    a->ring = 1;
    a->ring_dma = 1;
    a->pipelined = d == 64;
    a->heads_per_wg = 1;
    a->same_head = 0;
    a->n_units = (int)units;
    a->units_per_xcd = (a->n_units + 7) / 8;
    a->xcd_period = 0;
    // Of the workgroups that share a compute unit the oldest goes first, so that the last ones of a launch would end
    // alone, at the pace of a single wavefront (1 us per tile; 19 wavefronts on a unit do a tile in 0.09).  From this
    // workgroup on, the last that fit the chip together, wavefronts give way the further they have come (the kernel's
    // s_setprio): 256 pairs of 577 tokens 22.6 -> 20.9 us, 64 pairs of 2100 with 32 features 69.8 -> 64.0.  Not for
    // all of several rounds: 64 pairs of 2100, tiles of 128, 65.1 -> 76.8; nor for fewer than three wavefronts to a
    // SIMD, where there is nothing to share (32 pairs of 768 tokens, 32 features, 12.1 -> 12.4).
    // (To step down, wavefronts have to start above the default: for its whole length such a launch is issued ahead of what other
    // streams have on the same compute units.  Two layers at a time on two streams gain all the same: 64 pairs of 2100 beside 768 of
    // 197 63.7 us a pair of launches, 71.9 without priorities, 384 of 577 beside them 48.4 and 50.0; a 16 MiB elementwise kernel
    // beside 256 of 577 8.7 to 9.5 us both ways, beside 64 of 2100 10.7 to 11.7 and 7.8 to 10.1.)
    const long long grid = 8ll * a->units_per_xcd, last = (long long)resident * (a->n_cu > 0 ? a->n_cu : 256);
    a->ring_even_from = resident * waves < 9 ? (int)grid : grid > last ? (int)(grid - last) : 0;
    return 1;
}

// LDS bytes of the windowed-attention kernel: the table (rounded up to 1 KiB) and, per wavefront
// (two to a stream), two sets of V, K and 32 query rows (5 KiB each).
size_t qflash_win_lds_bytes(int streams, int table_bytes) {
    return (((size_t)table_bytes + 1023) & ~(size_t)1023) + (size_t)streams * 2 * 2 * 5120;
}

size_t qflash_win_dyn_lds_bytes(int streams, int table_bytes) {
    return (((size_t)table_bytes + 1023) & ~(size_t)1023) + (size_t)streams * kWinDynSets * (kWinDynSetBytes + 8) + 8 + kDynConstBytes;
}

static int plan_win(int d, int kv_tile, int lds_limit, int table_bytes, int max_streams, size_t (*lds_bytes)(int, int), QflashKernelArgs* a) {
    (void)kv_tile;                      // a single KV tile either way: 64 and 128 give the same result
    a->win_mode = 0;
    if (d != 32 || a->N <= 32 || a->N > 64 || a->per_head || a->qmax) return 0;
    if (a->bias && (a->bias_B < 1 || a->bias_H < 1 || a->B % a->bias_B != 0 || a->H % a->bias_H != 0)) return 0;
    const long long T = (long long)a->B * a->H;
    const int cus = a->n_cu > 0 ? a->n_cu : 256;
    // as many runs as there are pairs, up to max_streams per compute unit (fewer where the table leaves
    // less LDS); equal shares
    while (max_streams > 0 && lds_bytes(max_streams, table_bytes) > (size_t)lds_limit) --max_streams;
    if (max_streams == 0) return 0;
    long long runs = T < (long long)max_streams * cus ? T : (long long)max_streams * cus;
    const long long chunk = (T + runs - 1) / runs;
    runs = (T + chunk - 1) / chunk;
    int streams = (int)((runs + cus - 1) / cus);
    if (streams > max_streams) streams = max_streams;
    const long long groups = (runs + streams - 1) / streams;
    if (chunk >= (1ll << 30) || groups >= (1ll << 30)) return 0;
    if (lds_bytes(streams, table_bytes) > (size_t)lds_limit) return 0;
    a->win_mode = 1;
    a->win_streams = streams;
    a->win_chunk = (int)chunk;
    a->win_groups = (int)groups;
    a->win_table_lds = (table_bytes + 1023) & ~1023;
    return 1;
}

int qflash_plan_win(int d, int kv_tile, int lds_limit, int table_bytes, QflashKernelArgs* a) {
    return plan_win(d, kv_tile, lds_limit, table_bytes, 8, qflash_win_lds_bytes, a);
}

int qflash_plan_win_dynamic(int d, int kv_tile, int lds_limit, QflashKernelArgs* a) {
    return plan_win(d, kv_tile, lds_limit, kTableMaxBytes, kWinDynStreams, qflash_win_dyn_lds_bytes, a);
}

void qflash_win_order(QflashKernelArgs* a) {
    const bool has_bias = a->bias || a->dyn_mask;
    const int bias_B = has_bias ? a->bias_B : 1, bias_H = has_bias ? a->bias_H : 1;
    a->win_rb = a->B / bias_B;
    a->win_rh = a->H / bias_H;
    a->win_inv_r = qflash_reciprocal((unsigned)a->win_rb * (unsigned)a->win_rh);
    a->win_inv_rh = qflash_reciprocal((unsigned)a->win_rh);
    a->win_inv_bh = qflash_reciprocal((unsigned)bias_H);
}

// LDS bytes of the kernel that shares out the keys: the table (rounded up to 1 KiB), one part of P V
// per wavefront, row maxima, row sums and alpha (32 x 20 words each).
size_t qflash_split_lds_bytes(int d, int waves, int table_bytes) {
    return (((size_t)table_bytes + 1023) & ~(size_t)1023) + (size_t)waves * 128 * (size_t)d + 4 * 32 * 3 * 20;
}

int qflash_plan_split(int d, int lds_limit, int table_bytes, QflashKernelArgs* a) {
    a->split_waves = 0;
    if (a->qmax) return 0;
    const int nblk = (a->N + 31) / 32;
    const long long units = (long long)a->B * a->H * nblk;
    const int cus = a->n_cu > 0 ? a->n_cu : 256;
    // Where the line lies (d = 64, one image to a small batch, us per launch here against the other kernels):
    // N = 197: 336 units 5.7 / 8.1, 672 units 8.3 / 8.2; N = 577: 456 units 10.1 / 12.7, 912 units 17.7 / 12.9;
    // N = 1025: 396 units 14.8 / 19.6, 792 units 26.5 / 19.8.  One KV tile (N = 64) has no chain to cut:
    // 192 units 3.7 / 3.9, 384 units 4.2 / 3.9.  The windowed kernel is as fast from the start.
    if (a->win_mode || units > (nblk > 2 ? 2ll : 1ll) * cus) return 0;
    // Two blocks per wavefront make one KV tile of 64 keys local to it and halve what the chain reads; one
    // tile in all is spread over two wavefronts (49 tokens with a bias: 3.8 against 4.5 us).  Eight
    // wavefronts while every workgroup has a compute unit to itself, else four so that two fit one
    // (N = 577, 456 units: 10.1 against 13.2 us); parts of 32 features are half the size.
    const int kb = nblk > 2 ? 2 : 1;
    const int parts = (nblk + kb - 1) / kb;
    const int waves = parts > 4 && units * d <= 64ll * cus ? 8 : 4;
    // The table (up to 40 KiB per workgroup) pays once a wavefront looks up more than it fetches.
    const int table = nblk > 2 ? (table_bytes + 1023) & ~1023 : 0;
    if (qflash_split_lds_bytes(d, waves, table) > (size_t)lds_limit) return 0;
    a->split_waves = waves;
    a->split_blocks = kb;
    a->split_table_lds = table;
    a->split_qtiles_inv = (unsigned)((((unsigned long long)1 << 32) + nblk - 1) / nblk);   // (not used where nblk is 1)
    a->n_qtiles = nblk;
    a->n_units = (int)units;
    a->units_per_xcd = (int)((units + 7) / 8);
    a->xcd_period = 0;
    return waves;
}

// The kernel a call takes, but for launches too small to fill the chip (qflash_plan_split).
int qflash_plan_family(int d, int kv_tile, int lds_limit, QflashCallKind kind, int* table_bytes, QflashKernelArgs* a) {
    const int BH = a->B * a->H, N = a->N;
    if (qflash_plan_fwd(BH, N, d, kv_tile, lds_limit, a) != 0) return -1;
    a->split_waves = 0;
    a->win_mode = 0;
    a->cu_mode = 0;
    // Room for a table that is made on the GPU, its size unknown here (a larger one is not used then, although the
    // quantising kernel has built it): any table, but for rings of 64 features and tile 64 24 KiB, so that four workgroups
    // share a compute unit, not two (128 pairs of 1025 tokens from float32 104.5 -> 92.5 us; 107 instead of 106 where the
    // table does not fit).  N(0,1) inputs fit it if their largest magnitudes reach 5.04 (geometric mean of Q's and K's):
    // from about two million elements on; the finer scales of smaller tensors compute their weights.  For
    // rings of 32 features 32 KiB (three quarters of the variance, four workgroups), and never more than the
    // workgroup moves anyway (1728 windows of 144 tokens 82.3 -> 77.9 us with a table of 18 KiB).
    if (kind.on_device && *table_bytes > 0) {
        int room = kTableMaxBytes;
        if (a->ring_dma) { if (kv_tile == 64) room = 24 * 1024; }
        else if (d == 32 && N > 64 && !a->bias) room = 32 * 1024;
        else if (a->resident && 4ll * a->heads_per_wg * N * d < room) room = 4 * a->heads_per_wg * N * d & ~1023;
        *table_bytes = room;
    }
    const int table = *table_bytes;
    if (kind.from_floats) {
        if (a->bias || a->dyn_mask) (void)qflash_plan_win_dynamic(d, kv_tile, lds_limit, a);
    } else if (!a->qmax && qflash_plan_win(d, kv_tile, lds_limit, table, a) == 0 && table > 0) {
        (void)qflash_plan_win(d, kv_tile, lds_limit, 0, a);
    }
    (void)qflash_plan_ring(d, lds_limit, table, a);
    if (kind.from_floats) {
        if (!a->win_mode) (void)qflash_plan_cu_dynamic(BH, N, d, kv_tile, lds_limit, a);
    } else if (!a->qmax && !a->win_mode && !kind.on_device) {          // (the whole-compute-unit kernel exists for Algorithm 1 only)
        auto plan = [&](int bytes) {
            return kv_tile == 64 ? qflash_plan_cu(BH, N, d, kv_tile, lds_limit, bytes, a) : qflash_plan_cu128(BH, N, d, lds_limit, bytes, a);
        };
        if (!plan(table) && table > 0) (void)plan(0);
        // (one pair per compute unit, tiles of 128 and no table, see qflash_attention_static: 192 pairs of 197 tokens
        // 9.1 us resident, 9.6 here)
        if (kind.static_table && a->cu_mode && kv_tile == 128 && a->cu_heads == 1) a->cu_mode = 0;
        if (a->per_head) (void)qflash_plan_cu_heads(BH, N, d, kv_tile, lds_limit, a);
    }
    return 0;
}

int qflash_plan_dynamic(int d, int kv_tile, int lds_limit, QflashKernelArgs* a, bool* fused, bool* wants_table) {
    if (qflash_plan_fwd(a->B * a->H, a->N, d, kv_tile, lds_limit, a) != 0) return -1;
    // Windows with a bias and short sequences (one that gives whole compute units to a workgroup) are quantised on the way in.
    *fused = a->bias && qflash_plan_win_dynamic(d, kv_tile, lds_limit, a) != 0;
    if (!*fused) (void)qflash_plan_win(d, kv_tile, lds_limit, 0, a);
    // a launch whose keys are shared out computes its weights (building a table takes longer than it saves)
    *wants_table = qflash_plan_split(d, lds_limit, 0, a) == 0;
    *fused = *fused || (*wants_table && qflash_plan_cu_dynamic(a->B * a->H, a->N, d, kv_tile, lds_limit, a) != 0);
    return 0;
}

int qflash_kernel_family(const QflashKernelArgs& a) { return a.win_mode ? 4 : a.cu_mode ? 3 : a.ring ? 2 : a.resident ? 1 : 0; }

void qflash_plan_report(const QflashKernelArgs& a, int d, qflash_plan_info* out) {
    out->kernel = qflash_kernel_family(a);
    if (out->kernel == 4) {
        out->pairs_per_workgroup = a.win_streams * a.win_chunk;
        out->wavefronts_per_pair = 2;
        out->query_blocks = 2;
        out->units = out->workgroups = a.win_groups;
    } else if (out->kernel == 3) {
        out->pairs_per_workgroup = a.cu_heads;
        out->wavefronts_per_pair = a.cu_waves;
        out->query_blocks = (a.N + 31) / 32;
        out->units = out->workgroups = a.cu_groups;
    } else {
        out->pairs_per_workgroup = a.heads_per_wg;
        out->wavefronts_per_pair = a.waves_per_head;
        out->query_blocks = a.n_qtiles;
        out->units = a.n_units;
        out->workgroups = 8 * a.units_per_xcd;
        out->tile_by_tile = a.ring_dma || (a.resident && a.pipelined && d == 64 && (a.kv_tile == 64 || a.N > 256)) ? 1 : 0;
        out->bias_period_units = a.xcd_period;
        out->units_per_xcd = a.units_per_xcd;
    }
}
