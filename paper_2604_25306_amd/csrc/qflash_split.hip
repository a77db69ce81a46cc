// gfx950 kernel of the integer-only fused attention forward pass (Algorithm 1) for launches too small
// to fill the chip: the keys of a block of query rows are shared out to the wavefronts of a workgroup.
//
// Every other kernel here gives a wavefront 32 query rows and lets it walk over the KV tiles one
// after the other, about 1 us per tile for a wavefront on its own.  With a few images the chip has
// more SIMDs than there are such wavefronts, and the time of the launch is that serial chain.  Here a
// workgroup serves 32 query rows of one (batch, head) pair and wavefront w takes the keys
// [32 w, 32 w + 32) of a chunk of 32 W keys.  Algorithm 1 is sequential in the KV tiles only through
// the running maximum and through ScaleRelease of what has been accumulated, and both are cheap:
//   1. every wavefront computes its 32 x 32 scores and their row maxima and leaves the maxima in LDS;
//   2. (barrier) every wavefront reads the maxima of the whole chunk; the running maximum before and
//      after its own tile is a prefix maximum of them.  With it the weights of its keys, their sum,
//      its 32 keys' part of P V (int32, to LDS) and, one wavefront per tile, alpha are all local;
//   3. (barrier) the chain over the tiles, l <- floor(l alpha) + sum, O <- floor(O alpha) + P V, runs
//      over a different split of the data: every lane owns four features of one row and walks over
//      the tiles of the chunk, a multiply-high and two or three additions per tile and feature.
// The order of the operations on every (l, O) is exactly that of Algorithm 1 (the part of P V that a
// tile contributes is an exact integer sum in any order), so the bits are those of the other kernels.
//
// What bounds it: the latency of one pass (kernel arguments, operand loads, two products, the weights,
// two barriers: about 3.5 us of launch included) and, as the launch grows, vector issue: the prologue,
// the chain and the normalisation are paid per 32 query rows and make it two to three times the vector
// instructions of a wavefront that walks over its tiles alone.  K, Q and the bias go straight to
// operand registers; V passes through LDS for its transposing read, in the place its wavefront's part
// of P V takes afterwards.  Two 32-key blocks per wavefront rather than one: a tile of 64 keys is then
// local to a wavefront and the chain reads half as many parts.  The weight table, where it is used,
// lands in LDS by direct loads beside the operands (four to a setting of M0: +0.1 us instead of +0.3).
// Measured (us per launch, HIP graph, before -> after): N = 197, 3 pairs 7.9 -> 4.5 (4.2 with the short arguments), 48 pairs 8.1 -> 5.7;
// N = 577, 12 pairs 12.6 -> 7.4; N = 1025, 3 pairs 19.7 -> 10.0; d = 32, N = 1000, 4 pairs 25 -> 7.7.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "qflash_launch.h"
#include "qflash_tile.h"

namespace {

// (M0 is written by the direct loads of the table and declared as clobbered)
#pragma clang diagnostic ignored "-Winline-asm"

extern __shared__ __align__(1024) int8_t smem_split[];

constexpr int kRowPitch = 20;      // words per query row of the tables of row maxima, row sums and alpha (16 used):
                                   // 16-byte reads of eight neighbouring rows fall into different banks

// Row of the quad (q, g) of features 8 q + 4 g .. + 3 in a part of P V: permuted, so that the chain,
// whose lanes read many quads of one row, meets different banks.
__device__ __forceinline__ int part_offset(int q, int g, int row) { return 1024 * q + 512 * g + 16 * (row ^ ((q + 4 * g) & 7)); }

// (batch, head) pair of a unit = unit / n_qtiles, with the reciprocal made on the host.
__device__ __forceinline__ int split_pair(const QflashLaunchArgs& a, int unit) {
    return a.n_qtiles == 1 ? unit : (int)__umulhi((unsigned)unit, a.split_qtiles_inv);
}

// KB: 32-key blocks per wavefront (1 or 2).
template <int D, int BC, int BIAS, int XM, int KB, class Args>
__device__ __forceinline__ void split_body(const Args& a) {
    constexpr bool KZ = XM == kExpShift0;
    constexpr bool SB = XM == kExpTable && !BIAS;   // scores (and maxima) carry the offset 2^30
    constexpr int kExcluded = SB ? kMaskedBiased : kNegBig;
    constexpr int KSTEPS = D / 32, TB = D / 32;
    constexpr int WPT = BC / 32 / KB;               // wavefronts (parts) per KV tile
    constexpr int kPart = 32 * D * 4;               // bytes of one wavefront's part of P V
    constexpr int FPL = 4 * KB;                     // chain: features per lane
    constexpr int kLanesPerRow = D / FPL;           // chain: lanes per query row
    constexpr int kRowsPerPass = 64 / kLanesPerRow; // chain: rows a wavefront serves at a time
    constexpr int kPasses = 32 / kRowsPerPass;      // chain: such groups of rows, shared out to the wavefronts
    constexpr int kMine = kPasses > 4 ? kPasses / 4 : 1;   // at most, with at least four wavefronts

    const int unit = (int)(blockIdx.x & 7) * a.units_per_xcd + (int)(blockIdx.x >> 3);
    if (unit >= a.n_units) return;
    const int N = a.N;
    const int bh = split_pair(a, unit);
    const int rb = unit - bh * a.n_qtiles;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = (int)(blockDim.x >> 6);           // a multiple of 4
    const int g = lane >> 5, li = lane & 31;
    const int row0 = 32 * rb;
    const size_t head_off = (size_t)bh * N * D;
    const int8_t* Qh = a.Q + head_off;
    const int8_t* Kh = a.K + head_off;
    const int8_t* Vh = a.V + head_off;
    const int nblk = (N + 31) >> 5;                 // 32-key blocks of the sequence

    // ---- operand loads.  Rows beyond the sequence read the last one (their weights are 0, or their
    //      results are never stored).  (Uniform base plus a 32-bit lane offset.)
    v4i qreg[KSTEPS], kreg[KB][KSTEPS], vreg[KB][TB];
    {
        const unsigned off = (unsigned)(min(row0 + li, N - 1) * D + 16 * g);
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) qreg[s] = *(const v4i*)(Qh + off + 32 * s);
    }
    auto load_k = [&](int blk) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const unsigned off = (unsigned)(min(32 * (blk + kb) + li, N - 1) * D + 16 * g);
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) kreg[kb][s] = *(const v4i*)(Kh + off + 32 * s);
        }
    };
    // V block: 16-byte pieces in row-major order, piece `lane` (and 64 + lane)
    auto load_v = [&](int blk) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int s = 0; s < TB; ++s) {
                const int x = 64 * s + lane, r = x / (D / 16), pc = x % (D / 16);
                vreg[kb][s] = *(const v4i*)(Vh + (unsigned)(min(32 * (blk + kb) + r, N - 1) * D + 16 * pc));
            }
    };
    if (KB * wave < nblk) {
        load_k(KB * wave);
        load_v(KB * wave);
    }
    const QflashHeadConsts hc = head_consts(a, bh);
    const ExpConst<> c = make_exp_const(hc);
    // ---- LDS: [weight table][one part per wavefront: V, then its part of P V][row maxima][row sums][alpha];
    //      the dynamic LDS is the only LDS of the kernel, so the table index is its address
    const int lds0 = (int)(size_t)(lds_void)smem_split;
    const int tbytes = XM == kExpTable ? a.split_table_lds : 0;
    if (XM == kExpTable)
        for (int it = 4 * wave, n = (hc.lut_bytes + 1023) >> 10; it < n; it += 4 * W) {
            const int8_t* src = (const int8_t*)hc.lut + 1024 * it;
            if (it + 4 <= n) load_4k_to_lds(src, 16 * lane, lds0 + 1024 * it);
            else
                for (int x = it; x < n; ++x, src += 1024) load_1k_to_lds(src, 16 * lane, lds0 + 1024 * x);
        }
    int8_t* parts = smem_split + tbytes;
    int8_t* part = parts + wave * kPart;
    int* maxs = (int*)(parts + W * kPart);                                     // [32 rows][kRowPitch]
    int* sums = maxs + 32 * kRowPitch;                                         // likewise
    int* alphas = sums + 32 * kRowPitch;                                       // [32 rows][kRowPitch]
    // Where the pieces of V go in LDS: permuted by the row as everywhere (swizzled_lane_offsets).
    auto store_v = [&]() {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int s = 0; s < TB; ++s) {
                const int x = 64 * s + lane, r = x / (D / 16), pc = x % (D / 16);
                *(v4i*)(part + 32 * D * kb + r * D + 16 * (pc ^ ((r >> 2) & (D / 16 - 1)))) = vreg[kb][s];
            }
    };
    const int v_lane = swizzled_lane_offsets<D>(lane).v_off;
    const int part_addr = lds0 + tbytes + wave * kPart;

    const int32_t* bias_row = nullptr;
    if (BIAS) bias_row = bias_lane_base(a, bh, row0, row0 + li, li, g);

    // ---- the chain's share of this wavefront: passes wave, wave + W, ...; lane (row cr of the pass, FPL features)
    const int cr = lane / kLanesPerRow, cj = lane % kLanesPerRow;
    v4i o[kMine][KB];
    int l[kMine];
#pragma unroll
    for (int p = 0; p < kMine; ++p) {
#pragma unroll
        for (int q = 0; q < KB; ++q) o[p][q] = v4i{kAccBias, kAccBias, kAccBias, kAccBias};
        l[p] = 0;
    }

    int carry = SB ? kMInit + kAccBias : kMInit;    // running maximum of row li before this chunk
    const int t_mine = wave / WPT;                  // tile of this wavefront within a chunk
    for (int blk0 = 0; blk0 < nblk; blk0 += KB * W) {
        const int blk = blk0 + KB * wave;
        const bool active = blk < nblk;
        const int n_here = min(W, (nblk - blk0 + KB - 1) / KB);     // parts of this chunk
        const bool more = blk + KB * W < nblk;
        v16i s[KB];
        int mx = kExcluded;
        if (active) {
            // ---- step 1 and the bias; keys beyond the sequence fall out
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                s[kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kreg[kb][0], qreg[0], SB ? offset_block() : v16i{0}, 0, 0, 0);
#pragma unroll
                for (int ks = 1; ks < KSTEPS; ++ks) s[kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kreg[kb][ks], qreg[ks], s[kb], 0, 0, 0);
            }
            if (more) load_k(blk + KB * W);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const int n_valid = N - 32 * (blk + kb);        // may be <= 0 for the second block
                if (BIAS == kBiasPacked) {
                    if (n_valid > 0) {
#pragma unroll
                        for (int a4 = 0; a4 < 4; ++a4) {
                            const v4i bv = *(const v4i*)(bias_row + (size_t)(4 * (blk + kb) + a4) * 256);
#pragma unroll
                            for (int b = 0; b < 4; ++b) s[kb][4 * a4 + b] = __builtin_elementwise_add_sat(s[kb][4 * a4 + b], bv[b]);
                        }
                    } else {
#pragma unroll
                        for (int v = 0; v < 16; ++v) s[kb][v] = kExcluded;
                    }
                } else if (BIAS == kBiasPlain && n_valid >= 32) {
#pragma unroll
                    for (int a4 = 0; a4 < 4; ++a4) {
                        const v4i_a4 bv = *(const v4i_a4*)(bias_row + 32 * (blk + kb) + 8 * a4 + 4 * g);
#pragma unroll
                        for (int b = 0; b < 4; ++b) s[kb][4 * a4 + b] = __builtin_elementwise_add_sat(s[kb][4 * a4 + b], bv[b]);
                    }
                } else if (BIAS == kBiasPlain) {
#pragma unroll
                    for (int a4 = 0; a4 < 4; ++a4)
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const int col = 8 * a4 + 4 * g + b;
                            const int bv = col < n_valid ? bias_row[32 * (blk + kb) + col] : INT32_MIN;
                            s[kb][4 * a4 + b] = __builtin_elementwise_add_sat(s[kb][4 * a4 + b], bv);
                        }
                } else if (n_valid < 32) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (8 * (v >> 2) + 4 * g + (v & 3) >= n_valid) s[kb][v] = kExcluded;
                }
            }
            // ---- step 2
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int v = 0; v < 16; v += 2) mx = max(max(mx, s[kb][v]), s[kb][v + 1]);
            const HalfPair hp = both_halves(mx);
            mx = max(hp.x, hp.y);
        }
        if (g == 0) maxs[li * kRowPitch + wave] = mx;
        if (XM == kExpTable && blk0 == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's share of the table
        __syncthreads();
        // ---- step 3: running maximum before and after this wavefront's tile, and after the chunk
        int m_old = carry, m_new = carry;
        {
            int run = carry;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * q < W) {
                    const v4i mm = *(const v4i*)(maxs + li * kRowPitch + 4 * q);
#pragma unroll
                    for (int t = 0; t < 4 / WPT; ++t) {
                        const int tile = q * (4 / WPT) + t;
                        if (tile == t_mine) m_old = run;
#pragma unroll
                        for (int w = 0; w < WPT; ++w) run = max(run, mm[WPT * t + w]);
                        if (tile == t_mine) m_new = run;
                    }
                }
            carry = run;
        }
        int rowsum = 0;
        if (active) {
            store_v();
            if (more) load_v(blk + KB * W);
            const int lo = m_new + c.x_floor, ml = m_new - c.lead;
            // ---- step 4 (one wavefront per tile)
            if (wave % WPT == 0) {
                const int a_hat = shift_exp2<KZ>(max(m_old, lo), m_new, ml, c);
                if (g == 0) alphas[li * kRowPitch + t_mine] = (int)min(((unsigned)a_hat * (unsigned)hc.a_mul) >> 14, 65536u);
            }
            // ---- steps 5 to 7
            v4i pk[KB];
            if (XM == kExpTable) {
                const unsigned x_p = (unsigned)to_vgpr(hc.lut_xp), edge = (unsigned)m_new - x_p;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        s[kb][v] = table_weight(SB ? __builtin_elementwise_sub_sat((unsigned)s[kb][v], edge)
                                                   : __builtin_elementwise_sub_sat(x_p, (unsigned)m_new - (unsigned)s[kb][v]));
            }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int a4 = 0; a4 < 4; ++a4) {
                    unsigned w;
                    if (XM == kExpTable) {
                        w = pack_weights((unsigned)s[kb][4 * a4], (unsigned)s[kb][4 * a4 + 1], (unsigned)s[kb][4 * a4 + 2], (unsigned)s[kb][4 * a4 + 3]);
                    } else {
                        unsigned pr[4];
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const int y = shift_exp2<KZ>(max(s[kb][4 * a4 + b], lo), m_new, ml, c);
                            pr[b] = c.weight(y);
                        }
                        w = pack_byte3(pr[0], pr[1], pr[2], pr[3]);
                    }
                    pk[kb][a4] = (int)w;
                    rowsum = add_bytes(w, rowsum);
                }
            const HalfPair hp = both_halves(rowsum);
            rowsum = hp.x + hp.y;
            // ---- step 8: this wavefront's part of P V
            v16i pv[TB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int t = 0; t < TB; ++t) {
                    const int va_addr = part_addr + 32 * D * kb + (v_lane ^ (32 * t));
                    const v2i_t lo2 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(size_t)va_addr);
                    const v2i_t hi2 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(size_t)(va_addr + 16 * D));
                    const v4i va = __builtin_shufflevector(lo2, hi2, 0, 1, 2, 3);
                    pv[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(va, pk[kb], kb == 0 ? v16i{0} : pv[t], 0, 0, 0);
                }
            // quad q = 4 t + a4 of lane (li, g): features 8 q + 4 g .. + 3 of row li
#pragma unroll
            for (int q = 0; q < 4 * TB; ++q) {
                const v4i w = {pv[q / 4][4 * (q % 4)], pv[q / 4][4 * (q % 4) + 1], pv[q / 4][4 * (q % 4) + 2], pv[q / 4][4 * (q % 4) + 3]};
                *(v4i*)(part + part_offset(q, g, li)) = w;
            }
        }
        if (g == 0) sums[li * kRowPitch + wave] = rowsum;
        __syncthreads();
        // ---- steps 9, 10: the chain over the tiles of the chunk
#pragma unroll
        for (int p = 0; p < kMine; ++p) {
            const int pass = wave + p * W;
            if (pass < kPasses) {
                const int r = pass * kRowsPerPass + cr;
                const int* al = alphas + r * kRowPitch;
                const int* su = sums + r * kRowPitch;
                const int8_t* src[KB];
#pragma unroll
                for (int q = 0; q < KB; ++q) src[q] = parts + (KB == 1 ? part_offset(cj >> 1, cj & 1, r) : part_offset(cj, q, r));
                for (int w0 = 0; w0 < n_here; w0 += WPT) {
                    const ReleaseConst rel = make_release((unsigned)*al++);
                    l[p] = release_l(l[p], rel);
#pragma unroll
                    for (int q = 0; q < KB; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[p][q][e] = release_acc(o[p][q][e], rel);
#pragma unroll
                    for (int b = 0; b < WPT; ++b) {
                        if (w0 + b < n_here) {
                            l[p] += *su;
#pragma unroll
                            for (int q = 0; q < KB; ++q) o[p][q] += *(const v4i*)src[q];
                        }
                        ++su;
#pragma unroll
                        for (int q = 0; q < KB; ++q) src[q] += kPart;
                    }
                }
            }
        }
        // (the next chunk writes its maxima, which the chain does not read, then meets a barrier before
        // anything the chain reads is written again)
    }
    // ---- step 11
#pragma unroll
    for (int p = 0; p < kMine; ++p) {
        const int pass = wave + p * W;
        const int i = row0 + pass * kRowsPerPass + cr;
        if (pass < kPasses && i < N) {
            int8_t* dst = a.O + head_off + (unsigned)(i * D + FPL * cj);
            unsigned w[KB];
            normalise_quads<20, KB>(o[p], l[p], a.out_round != 0, w);
            if (KB == 1) *(unsigned*)dst = w[0];
            else *(v2i_t*)dst = v2i_t{(int)w[0], (int)w[KB - 1]};
        }
    }
}

// kExpAuto: per workgroup, table if the constants of its head have one (a.exp_mode of the launch).
template <int D, int BC, int BIAS, int XM, int KB, class Args>
__global__ __launch_bounds__(KB == 1 ? 1024 : 512) void qflash_fwd_split(const Args a) {
    if constexpr (XM == kExpAuto) {
        const int unit = (int)(blockIdx.x & 7) * a.units_per_xcd + (int)(blockIdx.x >> 3);
        if (unit >= a.n_units) return;
        if (head_consts(a, split_pair(a, unit)).lut_bytes > 0) split_body<D, BC, BIAS, kExpTable, KB>(a);
        else split_body<D, BC, BIAS, kExpShift, KB>(a);
    } else {
        split_body<D, BC, BIAS, XM, KB>(a);
    }
}

template <int D, int BC, int BIAS, int XM, int KB>
int launch_split(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    const unsigned grid = (unsigned)(8 * a.units_per_xcd), threads = (unsigned)(64 * a.split_waves);
    if (a.per_head) return qflash_launch_kernel<qflash_fwd_split<D, BC, BIAS, XM, KB, QflashKernelArgs>>(a, grid, threads, lds, lds_limit, st);
    return qflash_launch_kernel<qflash_fwd_split<D, BC, BIAS, XM, KB, QflashLaunchArgs>>(a, grid, threads, lds, lds_limit, st);
}

template <int D, int BC, int BIAS, int KB>
int launch_mode(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    if (a.exp_mode == kExpAuto) return launch_split<D, BC, BIAS, kExpAuto, KB>(a, lds, lds_limit, st);
    if (a.exp_mode == kExpTable) return launch_split<D, BC, BIAS, kExpTable, KB>(a, lds, lds_limit, st);
    if (a.exp_mode == kExpShift0) return launch_split<D, BC, BIAS, kExpShift0, KB>(a, lds, lds_limit, st);
    return launch_split<D, BC, BIAS, kExpShift, KB>(a, lds, lds_limit, st);
}

template <int D, int BC, int KB>
int launch_bias(const QflashKernelArgs& a, size_t lds, int lds_limit, hipStream_t st) {
    if (!a.bias) return launch_mode<D, BC, kBiasNone, KB>(a, lds, lds_limit, st);
    return a.bias_packed ? launch_mode<D, BC, kBiasPacked, KB>(a, lds, lds_limit, st) : launch_mode<D, BC, kBiasPlain, KB>(a, lds, lds_limit, st);
}

}  // namespace

int qflash_launch_fwd_split(const QflashKernelArgs& a, int d, int lds_limit, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    // everything the kernel's indexing assumes, checked once more where it is launched
    if (a.split_waves < 4 || a.split_waves % 4 != 0 || a.split_waves > 16 || a.qmax) return (int)hipErrorInvalidValue;
    if (a.n_qtiles != (a.N + 31) / 32 || (long long)a.n_qtiles * a.B * a.H != a.n_units || 8ll * a.units_per_xcd < a.n_units || a.xcd_period != 0)
        return (int)hipErrorInvalidValue;
    const bool table = a.exp_mode == kExpTable || a.exp_mode == kExpAuto;
    if (table && a.lut_bytes_max > a.split_table_lds) return (int)hipErrorInvalidValue;
    const size_t lds = qflash_split_lds_bytes(d, a.split_waves, table ? a.split_table_lds : 0);
    if (lds > (size_t)lds_limit) return (int)hipErrorInvalidValue;
    if ((a.split_blocks != 1 && a.split_blocks != 2) || a.split_waves * a.split_blocks > 16) return (int)hipErrorInvalidValue;
    if (d != 32 && d != 64) return (int)hipErrorInvalidValue;
    const bool wide = a.kv_tile == 128;
    if (a.split_blocks == 1) {
        if (d == 64) return wide ? launch_bias<64, 128, 1>(a, lds, lds_limit, st) : launch_bias<64, 64, 1>(a, lds, lds_limit, st);
        return wide ? launch_bias<32, 128, 1>(a, lds, lds_limit, st) : launch_bias<32, 64, 1>(a, lds, lds_limit, st);
    }
    if (d == 64) return wide ? launch_bias<64, 128, 2>(a, lds, lds_limit, st) : launch_bias<64, 64, 2>(a, lds, lds_limit, st);
    return wide ? launch_bias<32, 128, 2>(a, lds, lds_limit, st) : launch_bias<32, 64, 2>(a, lds, lds_limit, st);
}
