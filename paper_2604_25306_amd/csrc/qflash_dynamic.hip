// Dynamic per-tensor quantisation in front of the attention kernel (Eq. 1-2 evaluated on the fly,
// as in the paper's evaluation set-up), entirely on the GPU: no value ever travels to the host.
//
//   1. abs-max    max |x| over each of Q, K, V (float32): one partial maximum per workgroup (a
//                 maximum is exact in any order, so the result does not depend on the grid)
//   2. quantise   every workgroup finishes the reduction of its tensor; eight more workgroups derive the
//                 scales s_X = max|X| / 127 (double) and, from s_Q and s_K, every integer constant of
//                 the attention kernel -- the same routine the host entry point uses -- and build
//                 the weight table of those constants if it is at most 40 KiB.  The others compute
//                 x_hat = clip(rint(x * r), -127, 127), r = float32(127) / max|x|: one float32
//                 division per tensor, one float32 multiplication and one round-half-to-even per
//                 element (the precision the rounding decision is defined in)
//   2b. bias      (optional) a bias in real units and an exclusion mask are brought to the integer
//                 score unit of the scales just found and written in the packed layout
//   3. attention  the usual kernel, reading its constants from the device structure of step 2
// (The whole-compute-unit kernel, see qflash_cu.hip, takes over steps 2 and 3 from the partial maxima on, the
// windowed one with a bias, see qflash_win.hip, also step 2b.)
//
// Steps 1 and 2 stream the float32 tensors once each and are bound by HBM: 12 B read in step 1
// and 12 B read + 3 B written in step 2 per (q, k, v) element triple.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qflash.h"
#include "qflash_internal.h"
#include "qflash_derive_device.h"

namespace {

constexpr int kDynThreads = 512;
constexpr int kDynMaxPartials = 256;     // workgroups per tensor at most: one partial maximum per thread of half a workgroup
constexpr int kTableWgs = 8;             // workgroups that build the weight table, beside the streaming ones

// Maximum over the workgroup (512 threads); every thread gets the result.
__device__ __forceinline__ float wg_reduce_max(float m, float* wmax /* 8 floats of LDS */) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    __syncthreads();                       // wmax may still be read from a previous call
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
    return fmaxf(fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3])),
                 fmaxf(fmaxf(wmax[4], wmax[5]), fmaxf(wmax[6], wmax[7])));
}

// grid.y = tensor (0: Q, 1: K, 2: V); n4 = elements / 4.  Each workgroup leaves its maximum in
// partial[tensor * gridDim.x + workgroup]: atomics on three words would serialise at the L2.
__global__ __launch_bounds__(kDynThreads) void qflash_dyn_absmax(const float* q, const float* k, const float* v,
                                                                 long long n4, float* partial) {
    __shared__ float wmax[8];
    const float* x = blockIdx.y == 0 ? q : blockIdx.y == 1 ? k : v;
    float m = 0.0f;
    for (long long i = (long long)blockIdx.x * kDynThreads + threadIdx.x; i < n4; i += (long long)gridDim.x * kDynThreads) {
        const v4f t = *(const v4f*)(x + 4 * i);
        m = fmaxf(fmaxf(m, fabsf(t[0])), fmaxf(fabsf(t[1]), fmaxf(fabsf(t[2]), fabsf(t[3]))));
    }
    m = wg_reduce_max(m, wmax);
    if (threadIdx.x == 0) partial[blockIdx.y * gridDim.x + blockIdx.x] = m;
}

// Maximum over n_partial <= kDynMaxPartials values by one workgroup; every thread gets the result.
__device__ __forceinline__ float wg_max(const float* partial, int n_partial, float* wmax /* 8 floats of LDS */) {
    return wg_reduce_max((int)threadIdx.x < n_partial ? partial[threadIdx.x] : 0.0f, wmax);
}

// grid.y = tensor, grid.x = n_partial streaming workgroups + those that make the constants; 4 elements per
// thread and iteration: 16 B in, 4 B out.  Every streaming workgroup first finishes the abs-max
// reduction of its tensor from the per-workgroup partial maxima (1 KB, L2-resident).
__global__ __launch_bounds__(kDynThreads) void qflash_dyn_quantize(const float* q, const float* k, const float* v,
                                                          int8_t* qo, int8_t* ko, int8_t* vo, long long n4,
                                                          const float* partial, int n_partial, double sqrt_d,
                                                          int out_round, QflashHeadConsts* hc, double* unit,
                                                          qflash_dynamic_info* info, uint8_t* table, int table_max) {
    __shared__ float wmax[8];
    __shared__ QflashHeadConsts sh_hc;
    // The workgroups beyond the streaming ones (tensor 0) do what needs all three maxima, while the others
    // stream: the first writes the scales and constants for the attention kernel that follows on the
    // stream; all of them derive the constants and, if there is room for one, build a share each of the
    // weight table.  (One workgroup of 256 threads took 10 to 15 us for it, longer than all the rest of
    // the kernel on tensors of up to a few million elements.)
    if (blockIdx.x >= (unsigned)n_partial) {
        if (blockIdx.y != 0) return;
        const int part = (int)blockIdx.x - n_partial, parts = (int)gridDim.x - n_partial;
        float a3[3];
        for (int t = 0; t < 3; ++t) a3[t] = wg_max(partial + t * n_partial, n_partial, wmax);
        if (threadIdx.x == 0) {
            derive_on_device(a3, sqrt_d, out_round, &sh_hc, part == 0 ? info : nullptr, part == 0 ? unit : nullptr);
            reserve_table(&sh_hc, table, table ? table_max : 0);
            if (part == 0) *hc = sh_hc;
        }
        __syncthreads();
        if (sh_hc.lut_bytes > 0) {
            const QflashHeadConsts h = sh_hc;
            const ExpConst<> c = make_exp_const(h);
            for (int i = part * kDynThreads + (int)threadIdx.x; i < h.lut_bytes; i += parts * kDynThreads)
                table[i] = (uint8_t)(i <= h.lut_xp ? table_entry(i, h.lut_xp, h, c) : 0u);
        }
        return;
    }
    const float* x = blockIdx.y == 0 ? q : blockIdx.y == 1 ? k : v;
    int8_t* y = blockIdx.y == 0 ? qo : blockIdx.y == 1 ? ko : vo;
    const float am = wg_max(partial + blockIdx.y * n_partial, n_partial, wmax);
    const float r = am == 0.0f ? 0.0f : __fdiv_rn(127.0f, am);
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (long long)n_partial * blockDim.x) {
        const v4f t = *(const v4f*)(x + 4 * i);
        unsigned w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float z = fminf(fmaxf(rintf(__fmul_rn(t[e], r)), -127.0f), 127.0f);
            w |= ((unsigned)(int)z & 0xffu) << (8 * e);
        }
        *(unsigned*)(y + 4 * i) = w;
    }
}

// Real bias and exclusion mask -> int32 bias in the lane-major packed layout the attention kernel
// reads (see qflash_pack_bias_kernel for the layout), in the score unit of the scales just found:
//   unit = (s_Q s_K) / sqrt(d),  b_hat = clip(floor(double(b) / unit + 0.5), -(2^20 - 1), 2^20 - 1)
// evaluated in float64 with one rounding per operation (the precision the decision is defined in).
// One thread per 16-byte word, i.e. four consecutive columns of a row: one load of four floats and one of
// four mask bytes (neither needs more than element alignment; 12.9 us for 2 M elements with single
// loads and a reduction of the maxima in every workgroup).
typedef float v4f_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32_a1 __attribute__((aligned(1)));
__global__ __launch_bounds__(256) void qflash_dyn_bias(const float* __restrict__ bias, const uint8_t* __restrict__ mask,
                                                      int32_t* __restrict__ packed, int N, long long n_words,
                                                      const double* __restrict__ unit_p) {
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= n_words) return;
    const double unit = *unit_p, inv = 1.0 / unit;
    const int nb = (N + 31) / 32;
    const int lane = (int)(t & 63), a4 = (int)((t >> 6) & 3);
    const unsigned blk = blockIdx.x;                       // 256 words: one 32 x 32 block
    const int cb = (int)(blk % nb);
    const unsigned sr = blk / nb;
    const int rb = (int)(sr % nb);
    const long long slice = sr / nb;
    const int li = lane & 31, g = lane >> 5;
    const int row = min(32 * rb + li, N - 1), col0 = 32 * cb + 8 * a4 + 4 * g;
    const long long base = (slice * N + row) * (long long)N + col0;
    float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    unsigned mk = 0;
    if (col0 + 4 <= N) {
        if (bias) {
            const v4f_a4 w = *(const v4f_a4*)(bias + base);
            x[0] = w[0]; x[1] = w[1]; x[2] = w[2]; x[3] = w[3];
        }
        if (mask) mk = *(const u32_a1*)(mask + base);
    } else {
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (col0 + b < N) {
                if (bias) x[b] = bias[base + b];
                if (mask) mk |= (unsigned)mask[base + b] << (8 * b);
            }
    }
    int32_t w[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int32_t v = bias_word(x[b], unit, inv);
        w[b] = col0 + b < N && ((mk >> (8 * b)) & 0xffu) == 0 ? v : INT32_MIN;
    }
    *(int4*)(packed + 4 * t) = int4{w[0], w[1], w[2], w[3]};
}

}  // namespace

int qflash_launch_dynamic_bias(const float* bias, const uint8_t* mask, int slices, int N, int32_t* packed,
                               const double* unit, void* stream) {
    const long long n_words = qflash_packed_bias_words(slices, N);
    hipLaunchKernelGGL(qflash_dyn_bias, dim3((unsigned)((n_words + 255) / 256)), dim3(256), 0, (hipStream_t)stream, bias, mask,
                       packed, N, n_words, unit);
    return (int)hipGetLastError();
}

int qflash_dynamic_partials(long long n) {
    // enough workgroups to keep every HBM channel busy (one of eight wavefronts per compute unit and tensor);
    // each streams a grid-strided share
    long long wgs = (n / 4 + kDynThreads - 1) / kDynThreads;
    // (every workgroup of the second kernel re-reads all partial maxima of its tensor: with 2048
    // of them that prologue cost a fifth of the kernel)
    if (wgs > kDynMaxPartials) wgs = kDynMaxPartials;
    if (wgs < 1) wgs = 1;
    return (int)wgs;
}

int qflash_launch_absmax(const float* Qf, const float* Kf, const float* Vf, long long n, float* scratch, void* stream) {
    hipLaunchKernelGGL(qflash_dyn_absmax, dim3((unsigned)qflash_dynamic_partials(n), 3), dim3(kDynThreads), 0, (hipStream_t)stream, Qf, Kf, Vf,
                       n / 4, scratch);
    return (int)hipGetLastError();
}

int qflash_launch_dynamic_front(const float* Qf, const float* Kf, const float* Vf, int8_t* Qo, int8_t* Ko, int8_t* Vo,
                                long long n, double sqrt_d, int out_round, float* scratch,
                                QflashHeadConsts* hc_dev, double* unit, qflash_dynamic_info* info, uint8_t* table, int table_max,
                                void* stream) {
    hipStream_t st = (hipStream_t)stream;
    const long long n4 = n / 4;
    const int wgs = qflash_dynamic_partials(n);
    float* partial = scratch;         // 3 * wgs words
    const int rc = qflash_launch_absmax(Qf, Kf, Vf, n, partial, stream);
    if (rc != 0) return rc;
    hipLaunchKernelGGL(qflash_dyn_quantize, dim3((unsigned)wgs + (table ? kTableWgs : 1), 3), dim3(kDynThreads), 0, st, Qf, Kf, Vf,
                       Qo, Ko, Vo, n4, (const float*)partial, wgs, sqrt_d, out_round, hc_dev, unit, info, table, table_max);
    return (int)hipGetLastError();
}
