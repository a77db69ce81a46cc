// Internal interface between the host side of the C ABI and the gfx950 kernels.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "qflash.h"

#if defined(__HIPCC__)
#define QF_UNIT_HD __host__ __device__
#else
#define QF_UNIT_HD
#endif

// Integer constants of Algorithm 1 / 2 for one head, or for the whole tensor (see qflash_params).
struct QflashHeadConsts {
    int x_shift, s_inv, exp_mul, p_mul, p_shift, a_mul;
    // x_floor <= 0: score differences below it are clamped to it.  Chosen on the host so that
    // ShiftExp2 is exactly 0 at and below it, and every 32-bit intermediate is exact above it.
    int x_floor;
    // look-up mode (resident kernel only): table of int8 weights of these constants
    int lut_xp;              // table index = score - running max + lut_xp, clamped at 0
    int lut_bytes;           // bytes staged into LDS (multiple of 16)
    const uint8_t* lut;      // nullptr = none
};

// Per-head constants travel in the kernel arguments, which the host copies on every launch: packed, 20
// bytes per head (the unpacked structures made it 3.9 KB and 0.3 us).
constexpr int kQflashMaxParamHeads = 64;
constexpr int kTableMaxBytes = 40 * 1024;    // largest weight table, and the distance of two in the context's cache

struct QflashHeadWords {
    uint32_t w[5];   // s_inv | x_shift << 18 | p_shift << 22 | has table << 27; exp_mul; p_mul; a_mul; table slot | lut_xp << 8
};

// Arguments of a launch with one set of constants.
struct QflashLaunchArgs {
    const int8_t* Q;
    const int8_t* K;
    const int8_t* V;
    int8_t* O;
    const int32_t* bias;   // nullptr: no bias
    int bias_B, bias_H;
    int bias_packed;       // bias is in the lane-major layout written by qflash_launch_pack_bias
    int B, H, N;
    int out_round;
    // work decomposition: one unit = (batch*head, query tile); XCD x owns units
    // [x*units_per_xcd, (x+1)*units_per_xcd)
    int rows_per_wg, n_qtiles, n_units, units_per_xcd;
    int xcd_period;          // 0, or the number of units after which the bias slices repeat (a multiple of 8)
    int waves_per_head;      // wavefronts that serve one (batch, head) pair inside a workgroup
    int heads_per_wg;        // > 1 only when a pair fits one workgroup (n_qtiles == 1)
    int same_head;           // heads_per_wg > 1: the pairs of a workgroup are one head of consecutive batch elements
    unsigned split_qtiles_inv;   // kernel that shares out the keys of 32 query rows: ceil(2^32 / n_qtiles), unit / n_qtiles is the high word of the product
    int pipelined;           // resident only: K/V tiles are staged one ahead of their use
    int ring;                // pipelined only: LDS holds two KV tiles (in use / being staged), not the whole sequence
    int split_table_lds;     // that kernel: LDS bytes reserved for the weight table (a multiple of 1 KiB)
    int n_cu;                // compute units of the device if wave priority alternates by dispatch round, else 0
    // weight mode of the launch (uniform over heads): 2 = every head reads its table,
    // 1 = arithmetic with x_shift == 0 for every head, 0 = arithmetic, 3 = per workgroup: table if the
    // constants of its head have one (lut_bytes > 0), else arithmetic
    int exp_mode;
    int lut_bytes_max;       // LDS bytes reserved for the table: the largest of all heads
    // whole-compute-unit kernel (qflash_plan_cu): 1 if the launch takes it
    int cu_mode;
    int cu_heads;            // (batch, head) pairs per workgroup
    int cu_groups;           // workgroups
    int cu_waves;            // wavefronts per workgroup (at most 16)
    int cu_table_lds;        // LDS bytes reserved for the weight table (a multiple of 1 KiB)
    int cu_table_heads;      // per-head constants: number of heads with a table
    unsigned cu_inv_nblk, cu_inv_per, cu_inv_pairs, cu_inv_b;   // reciprocals (qflash_cu_reciprocals)
    // ring fed by direct global-to-LDS loads (no bias; set by qflash_plan_fwd and qflash_plan_ring): 1 if the launch takes it
    int ring_dma;
    int ring_table_lds;      // LDS bytes reserved for the weight table (a multiple of 1 KiB)
    int ring_even_from;      // workgroups from this index on give way to those behind them (qflash_plan_ring)
    // windowed-attention kernel (qflash_plan_win): 1 if the launch takes it
    int win_mode;
    int win_streams;         // pairs of wavefronts (one per half of the query rows) per workgroup, at most 8
    int win_chunk;           // consecutive pairs (in slice-major order) each pair of wavefronts works through
    int win_groups;          // workgroups
    int win_table_lds;       // LDS bytes reserved for the weight table (a multiple of 1 KiB)
    int win_rb, win_rh;      // replicas of a bias slice in batch and heads, and the reciprocals of their
    unsigned win_inv_r, win_inv_rh, win_inv_bh;   // product, the second and bias_H (qflash_win_order, qflash_divide)
    // where the attention kernel itself quantises (cu_mode or win_mode, and hc_dev, only; dyn_partial nullptr: it does not): Q, K and V are
    // float32, dyn_partial are the partial maxima of their magnitudes, dyn_partials per tensor, and the kernel derives the constants
    int dyn_partials;
    const float* dyn_partial;
    double dyn_sqrt_d;
    qflash_dynamic_info* dyn_info;           // may be null
    const uint8_t* dyn_mask;                 // win_mode: exclusion mask or null; bias is then float32 in real units, plain layout, or null
#ifdef QF_TRACE
    unsigned long long* trace;   // instrumented builds only: [workgroup][wavefront][16] timestamps
#endif
    // Constants computed on the GPU (dynamic quantisation): if set, the kernel reads this device
    // structure instead of the words below; exp_mode is then 0 (the host does not know the constants).
    const QflashHeadConsts* hc_dev;
    const uint8_t* lut_base;                 // table slot 0
    QflashHeadWords one;     // the constants if one set serves every head (hw[0] of QflashKernelArgs holds it too)
    int per_head;            // 0: it does; 1: head h uses hw[h] (H <= kQflashMaxParamHeads)
};

// Arguments of any launch: what the host plans and fills, and what kernels that serve per-head constants take.  Kernels
// that never do take the first part alone, since the host copies the arguments on every launch (1.7 KB and 0.3: 0.2 us a call).
struct QflashKernelArgs : QflashLaunchArgs {
    QflashHeadWords hw[kQflashMaxParamHeads];
    uint8_t cu_order[kQflashMaxParamHeads];   // cu_mode: the heads, those with a table first
    // read by the host alone
    int resident;            // 1: whole K/V of a head staged in LDS, 0: streamed per KV tile
    int kv_tile;             // KV tile size the plan was made for
    int qmax;                // 1: the quantised-maximum variant (not Algorithm 1 as printed; every x_shift must be 0)
    // kernel that shares out the keys of 32 query rows (qflash_plan_split): wavefronts per workgroup, 0 if not taken
    int split_waves;
    int split_blocks;        // 32-key blocks per wavefront: 1 or 2
    int device;              // the GPU of the launch (current when it is made)
};

#ifndef QF_TRACE
// What is read to find the constants lies in one line of 64 bytes, for either kind of arguments, and what the kernel that shares out
// keys needs to find its unit in the line of n_qtiles.  Each line more is waited for at the start, 0.1 us with the arguments in L2 and
// 0.3 when the host has just written them.  hw[0] apart from per_head: per-head launches of the ring (78 pairs of 618 tokens) 19.9 us a
// call against 19.7; split_qtiles_inv apart too: 3 pairs of 197 per head 4.75 and 6.1 a call against 4.64 and 5.7, 16 of 50 3.75 and 5.4
// against 3.65 and 5.1; `one` across two lines: 0.2 on every launch of the ring.
static_assert(offsetof(QflashLaunchArgs, hc_dev) % 64 == 0 && sizeof(QflashLaunchArgs) - offsetof(QflashLaunchArgs, hc_dev) + sizeof(QflashHeadWords) <= 64 &&
              offsetof(QflashLaunchArgs, split_table_lds) / 64 == offsetof(QflashLaunchArgs, n_qtiles) / 64, "order of the fields");
#endif

// n / d and n % d for 0 <= n < 2^32, d >= 1, with the reciprocal inv = floor((2^32 - 1) / d): the high word of n inv is the
// quotient or one less.  (Where n is the same for a wavefront nine scalar instructions, otherwise, as where the whole-compute-unit kernel
// deals out the pairs of heads, as many vector ones; the division is two dozen vector ones in a chain.)
QF_UNIT_HD inline unsigned qflash_reciprocal(unsigned d) { return 0xffffffffu / d; }
QF_UNIT_HD inline unsigned qflash_divide(unsigned n, unsigned d, unsigned inv, unsigned* rest) {
    unsigned q = (unsigned)(((unsigned long long)n * inv) >> 32), r = n - q * d;
    if (r >= d) { q += 1; r -= d; }
    *rest = r;
    return q;
}

// n / d for n d < 2^16, with the reciprocal inv = 2^16 / d + 1 (floor): two instructions.
QF_UNIT_HD inline unsigned qflash_small_reciprocal(unsigned d) { return 65536u / d + 1u; }
QF_UNIT_HD inline int qflash_small_quotient(int n, unsigned inv) { return (int)(((unsigned)n * inv) >> 16); }

// Number of bytes of a weight table that reaches down to -x_p (multiple of 16).
QF_UNIT_HD inline int qflash_table_bytes(int x_p) { return (x_p + 1 + 15) & ~15; }

// The constants of one head packed for the kernel arguments, and unpacked in the kernel.
inline QflashHeadWords qflash_pack_head(const QflashHeadConsts& h, int table_slot /* used if h has a table */) {
    QflashHeadWords r;
    const bool has = h.lut_bytes > 0;
    r.w[0] = (uint32_t)h.s_inv | (uint32_t)h.x_shift << 18 | (uint32_t)h.p_shift << 22 | (has ? 1u << 27 : 0u);
    r.w[1] = (uint32_t)h.exp_mul;
    r.w[2] = (uint32_t)h.p_mul;
    r.w[3] = (uint32_t)h.a_mul;
    r.w[4] = has ? (uint32_t)table_slot | (uint32_t)h.lut_xp << 8 : 0u;
    return r;
}
// x_floor of a set of constants: the smallest multiple of 2^-k at or below -20.5 octaves (qflash_fill_head_consts).
QF_UNIT_HD inline int qflash_x_floor(int s_inv, int x_shift) { return -((41 * s_inv + (2 << x_shift) - 1) >> (x_shift + 1)); }
QF_UNIT_HD inline QflashHeadConsts qflash_unpack_head(const QflashHeadWords& r, const uint8_t* lut_base) {
    QflashHeadConsts h;
    h.s_inv = (int)(r.w[0] & 0x3ffffu);
    h.x_shift = (int)(r.w[0] >> 18 & 15u);
    h.p_shift = (int)(r.w[0] >> 22 & 31u);
    h.exp_mul = (int)r.w[1];
    h.p_mul = (int)r.w[2];
    h.a_mul = (int)r.w[3];
    h.x_floor = qflash_x_floor(h.s_inv, h.x_shift);
    const bool has = (r.w[0] >> 27 & 1u) != 0;
    h.lut_xp = (int)(r.w[4] >> 8);
    h.lut_bytes = has ? qflash_table_bytes(h.lut_xp) : 0;
    h.lut = has ? lut_base + (size_t)(r.w[4] & 255u) * kTableMaxBytes : nullptr;
    return h;
}

// Which unit of work a workgroup takes (host and device: the kernels use it, qflash_plan_unit
// reports it).  Consecutive workgroup indices go to consecutive XCDs (each with its own L2), so XCD
// x = wg % 8 takes the units [x*units_per_xcd, (x+1)*units_per_xcd): neighbouring heads share an
// L2.  With a bias whose slices repeat every xcd_period units (windowed attention: the same windows
// in every image) XCD x instead takes the x-th eighth of every period, so that each L2 only ever
// sees an eighth of the bias.  The result may be >= n_units: such a workgroup has nothing to do.
QF_UNIT_HD inline int qflash_unit_of_workgroup(int wg, int units_per_xcd, int xcd_period) {
    const int x = wg & 7, k = wg >> 3;
    if (xcd_period == 0) return x * units_per_xcd + k;
    const int q = xcd_period >> 3;
    return (k / q) * xcd_period + x * q + k % q;
}

// Wavefronts per workgroup of the resident kernel (short sequences, N <= 256: 8, held to 128
// registers so that two workgroups share a compute unit; longer ones: 12), and of the streamed one.
constexpr int kResidentMaxWavesNarrow = 8;
constexpr int kResidentMaxWavesWide = 12;
constexpr int kStreamWaves = 4;
constexpr int kStreamRows = kStreamWaves * 32;

// Argument checks of the attention entry points (host only).  Returns QFLASH_OK or the error code.
int qflash_check_call(const void* Q, const void* K, const void* V, const void* O, const int32_t* bias, int bias_B,
                      int bias_H, bool bias_packed, int B, int H, int N, int d, int kv_tile, const qflash_params* p,
                      bool per_head, bool consts_on_device, bool qmax);

// LDS bytes of the resident kernel for `heads` pairs of N rows (ring_tile != 0: two KV tiles of that
// size instead of the whole sequence) plus a weight table; 0 if that exceeds lds_limit.  LDS bytes
// of the whole-compute-unit kernel.
size_t qflash_resident_lds_bytes(int N, int d, int heads, int table_bytes, int lds_limit, int ring_tile = 0);
size_t qflash_cu_lds_bytes(int N, int heads, int table_bytes);
// Wavefronts per workgroup of that kernel at most: with KV tiles of 128 it takes more than 128 registers, three wavefronts to a SIMD.
QF_UNIT_HD constexpr int qflash_cu_max_waves(int kv_tile) { return kv_tile == 64 ? 16 : 12; }

// Enqueue the forward kernel for head size d (32|64), KV tile (64|128).  Returns a hipError_t value.
int qflash_launch_fwd(const QflashKernelArgs& args, int d, int kv_tile, int lds_limit, void* stream);
// The same kernels instantiated for the quantised-maximum variant (called by qflash_launch_fwd when args.qmax).
int qflash_launch_fwd_qmax(const QflashKernelArgs& args, int d, int kv_tile, size_t lds_bytes, int lds_limit, int threads, void* stream);

// Choose the kernel variant for BH heads of N rows and fill the work decomposition fields
// (resident, pipelined, ring, ring_dma, rows_per_wg, waves_per_head, heads_per_wg, n_qtiles, n_units, units_per_xcd, xcd_period, same_head; reads bias, bias_B, B, H, per_head).
// Returns non-zero if the launch would be too large.
// lds_limit = LDS bytes one workgroup may use on this device.
int qflash_plan_fwd(int BH, int N, int d, int kv_tile, int lds_limit, QflashKernelArgs* args);   // n_cu is the caller's

// The kernel that gives a whole compute unit to one workgroup (short sequences, 64 features, tile 64,
// no bias, one set of constants): decides whether the launch takes it, assuming a weight table of
// table_bytes (0: none), and fills the cu_* fields.  Reads bias, per_head, n_cu (0: 256).  Returns cu_mode.
int qflash_plan_cu(int BH, int N, int d, int kv_tile, int lds_limit, int table_bytes, QflashKernelArgs* args);
// The same for KV tiles of 128.
int qflash_plan_cu128(int BH, int N, int d, int lds_limit, int table_bytes, QflashKernelArgs* args);
// The same kernel for per-head constants: heads whose table is at most cu_table_lds bytes (what is left of LDS)
// look their weights up, the others compute them.
int qflash_plan_cu_heads(int BH, int N, int d, int kv_tile, int lds_limit, QflashKernelArgs* args);
// The same kernel fed with float32 tensors (dynamic quantisation).
int qflash_plan_cu_dynamic(int BH, int N, int d, int kv_tile, int lds_limit, QflashKernelArgs* args);
constexpr int kCuDynExtraLds = 64;           // LDS of that variant beyond qflash_cu_lds_bytes
// Fills the reciprocals of such a launch: of the query blocks of a pair (qflash_small_quotient), of the 16-row pieces of a pair's three
// tensors (its kernel from float32), and, for qflash_divide, of the pairs and of B (its kernel for per-head constants).
void qflash_cu_reciprocals(QflashKernelArgs* args);
int qflash_launch_fwd_cu(const QflashKernelArgs& args, int lds_limit, void* stream);

// The persistent kernel for windowed attention (33 to 64 tokens, 32 features, one KV tile, no bias or a
// bias, packed or plain, whose extents divide B and H, one set of constants, Algorithm 1 only): decides
// whether the launch takes it and fills the win_* fields.  Reads bias, bias_B, bias_H, B, H, N, per_head,
// qmax, n_cu (0: 256).  Returns win_mode.
int qflash_plan_win(int d, int kv_tile, int lds_limit, int table_bytes, QflashKernelArgs* args);
void qflash_win_order(QflashKernelArgs* args);      // fills win_rb .. win_inv_bh of such a launch (reads bias, dyn_mask, bias_B, bias_H, B, H)
int qflash_launch_fwd_win(const QflashKernelArgs& args, int lds_limit, void* stream);
size_t qflash_win_lds_bytes(int streams, int table_bytes);
// The same kernel fed with float32 tensors (dynamic quantisation) and a bias in real units.
int qflash_plan_win_dynamic(int d, int kv_tile, int lds_limit, QflashKernelArgs* args);
size_t qflash_win_dyn_lds_bytes(int streams, int table_bytes);
constexpr int kWinDynStreams = 3;                 // runs of pairs per workgroup, four wavefronts each
constexpr int kWinDynSets = 4;                    // pairs in LDS per run
constexpr int kWinDynSetBytes = 6 * 1024;         // V, K, Q: 64 rows each
constexpr int kDynConstBytes = 44;                // constants and score unit, derived by the workgroup

// The kernel for launches that leave the chip idle, whose wavefronts share out the keys of 32 query rows:
// decides whether the launch, already planned for the other kernels, takes it, and then sets split_waves
// and replaces the work decomposition (n_qtiles, n_units, units_per_xcd, xcd_period).  table_bytes: weight
// table the call would use; split_table_lds says whether it is worth its room (0: compute the
// weights).  Reads B, H, N, n_cu, qmax and win_mode.  Returns split_waves.
int qflash_plan_split(int d, int lds_limit, int table_bytes, QflashKernelArgs* args);
int qflash_launch_fwd_split(const QflashKernelArgs& args, int d, int lds_limit, void* stream);
size_t qflash_split_lds_bytes(int d, int waves, int table_bytes);

// The whole choice of kernel, for a call with a->B, H, N, bias, bias_B, bias_H, per_head, qmax, dyn_mask and n_cu
// set: tries the plans above in the order the launch does and leaves one of win_mode, cu_mode, ring and resident
// set (none: streamed).  A launch and qflash_plan_query both go through it, so that the one cannot report what
// the other does not run.  *table_bytes: weight table the call would use, 0 none; with constants made on the GPU
// any positive number asks for one, and the room the launch keeps for it comes back.  qflash_plan_split decides
// afterwards whether the launch shares out keys instead.  Returns non-zero if the launch would be too large.
struct QflashCallKind {
    bool on_device;       // the integer constants are made on the GPU
    bool from_floats;     // the attention kernel itself quantises (qflash_plan_cu_dynamic, qflash_plan_win_dynamic)
    bool static_table;    // qflash_attention_static
};
int qflash_plan_family(int d, int kv_tile /* effective */, int lds_limit, QflashCallKind kind, int* table_bytes, QflashKernelArgs* args);
// Before that, for a call from float32 tensors (a->B, H, N, n_cu and, with a bias or mask, bias, bias_B, bias_H set):
// whether the attention kernel quantises on the way in, and whether a weight table is to be made at all.
int qflash_plan_dynamic(int d, int kv_tile /* effective */, int lds_limit, QflashKernelArgs* args, bool* fused, bool* wants_table);
// Kernel family of such a plan as in qflash_plan_info.kernel, and the decomposition it stands for.
int qflash_kernel_family(const QflashKernelArgs& args);
void qflash_plan_report(const QflashKernelArgs& args, int d, qflash_plan_info* out);
// A sequence of one KV tile gives the same result with either tile size; the smaller one's kernels need fewer registers.
inline int qflash_effective_tile(int kv_tile, int N) { return N <= 64 ? 64 : kv_tile; }

// The ring with direct global-to-LDS loads (long sequences, no bias, both Algorithm 1 and the
// quantised-maximum variant; work decomposition as for the ring of the resident kernel).
constexpr int kRingMaxWaves = 8;
int qflash_launch_fwd_ring(const QflashKernelArgs& args, int d, int lds_limit, void* stream);
size_t qflash_ring_lds_bytes(int waves, int kv_tile, int table_bytes, int d = 64);
// Slots in its LDS, each of one tile of K or V.
constexpr int qflash_ring_slots(int d) { return d == 64 ? 3 : 4; }
// Completes the plan of qflash_plan_fwd for that kernel: takes every sequence of 32 features without a bias and
// with more than one KV tile (planned as resident or streamed so far), and chooses the number of wavefronts
// per workgroup for a weight table of table_bytes.  Returns ring_dma.
int qflash_plan_ring(int d, int lds_limit, int table_bytes, QflashKernelArgs* args);

// GPUs per process for which per-device launch set-up is remembered.
constexpr int kQflashMaxDevices = 64;

// 1 if the resident kernel can also hold a weight table of table_bytes in LDS and copying it pays.
int qflash_table_fits(const QflashKernelArgs& args, int d, int table_bytes, int lds_limit);

// Enqueue the kernel that fills a weight table of n entries (n_padded bytes) for the constants hc.
int qflash_launch_build_table(uint8_t* tbl, int n, int n_padded, int x_p, const QflashHeadConsts& hc, void* stream);

// Bias in the lane-major layout the kernels read with 16-byte loads: number of 16-byte words for
// `slices` = bias_B * bias_H matrices of N x N, and the kernel that writes them from the plain layout.
long long qflash_packed_bias_words(int slices, int N);
int qflash_launch_pack_bias(const int32_t* bias, int slices, int N, int32_t* packed, void* stream);

// Enqueue the front end of the dynamic pipeline: abs-max of the three float32 tensors of n elements
// each (n a multiple of 4), derivation of the scales and constants into *hc_dev (and *info if not
// null) and of the real value of one score unit into *unit, quantisation into Qo, Ko, Vo.
// scratch: 3 * qflash_dynamic_partials(n) device floats.  The first step alone: qflash_launch_absmax.
int qflash_dynamic_partials(long long n);
int qflash_launch_absmax(const float* Qf, const float* Kf, const float* Vf, long long n, float* scratch, void* stream);
// table (may be null): room for a weight table of up to table_max bytes; if the table of the
// derived constants fits, the quantising kernel also builds it (a few workgroups more, beside the
// streaming ones) and records it in *hc_dev (lut, lut_bytes, lut_xp); lut_bytes == 0 says "none".
int qflash_launch_dynamic_front(const float* Qf, const float* Kf, const float* Vf, int8_t* Qo, int8_t* Ko, int8_t* Vo,
                                long long n, double sqrt_d, int out_round, float* scratch,
                                QflashHeadConsts* hc_dev, double* unit, qflash_dynamic_info* info, uint8_t* table, int table_max,
                                void* stream);
// Enqueue (after qflash_launch_dynamic_front on the same stream, same unit) the kernel that
// converts a real bias (float32 [slices,N,N] or null) and exclusion mask (uint8, same shape, or
// null) into the packed int32 bias of the scales found by the abs-max step.
int qflash_launch_dynamic_bias(const float* bias, const uint8_t* mask, int slices, int N, int32_t* packed,
                               const double* unit, void* stream);
