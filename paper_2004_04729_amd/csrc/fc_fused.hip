// Fully connected layers with few gradients in one launch: step size, mask, dither, codes and both products.  A code object of its own: no other call's
// kernels move.
#include <hip/hip_runtime.h>
#include "fc_direct_kernel.h"
#include "nsd_math.h"

namespace dbp {

// Every workgroup holds all codes in LDS: sixteen gradients a thread at most, while the first rows of its dense operand are on their way.  Step size: the tree of
// std_tree_kernel and std_finish_kernel (groups of 16 in order, level by level), codes: nsd_kernel's, so the results are the same bit for bit.  The first
// workgroup has no tile: it writes codes, statistics, bias gradient and step size.
// Bound by latencies: gradients, then codes and the dense operand, then the tile's own exchange.  A call, before / now (us): 64x100x10 with step
// size, mask and bias gradient 15.7 / 9.7, without 12.3 / 9.3 (the host's share of a call, from Python, is 9), 256x512x16 17.9 / 12.0, 512x4096x8 13.5 / 10.0, int8
// 128x1024x32 12.2 / 9.1, 64x784x128 12.1 / 9.1.
template <bool LAYER>
__global__ __launch_bounds__(64 * FCD_WAVES, 1) void fc_fused_kernel(FcdArgs a, FusedQuant q)
{
    extern __shared__ uint4 fcd_lds[];
    constexpr int NT = 64 * FCD_WAVES, PER = kFusedMax / NT;
    __shared__ __align__(16) int8_t s_codes[kFusedMax + 16];
    __shared__ float s_v[LAYER ? kFusedMax : 1], s_pair[2];
    __shared__ double s_sum[2][LAYER ? kFusedMax / 16 : 1];
    const int tid = threadIdx.x;
    const bool writer = blockIdx.x == 0;
    uint32_t nnz = 0, sat = 0, nonfinite = 0, top = 0;
    auto quantise = [&]() {
        float x[PER], m[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (i % 8 == 0 && NT * i >= q.n) break;                   // uniform
            const int e = min(tid + NT * i, q.n - 1);
            x[i] = q.delta[e];
            m[i] = LAYER && q.act ? q.act[e] : 1.0f;
        }
        float inv = q.inv_step;
        if constexpr (LAYER) {
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (i % 8 == 0 && NT * i >= q.n) break;
                const int e = tid + NT * i;
                x[i] = m[i] > 0.0f ? x[i] : 0.0f;
                if (e < q.n) s_v[e] = x[i];
            }
            __syncthreads();
            int have = q.n;                                          // values of the level below
            const int n0 = (have + 15) / 16;
            if (tid < n0) {
                float v[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) v[j] = s_v[min(16 * tid + j, have - 1)];
                double s1 = (double)v[0], s2 = (double)v[0] * (double)v[0];
#pragma unroll
                for (int j = 1; j < 16; ++j) {
                    const double d = (double)v[j];
                    if (16 * tid + j < have) { s1 += d; s2 = __builtin_fma(d, d, s2); }
                }
                s_sum[0][tid] = s1; s_sum[1][tid] = s2;
            }
            __syncthreads();
            double s1 = 0.0, s2 = 0.0;
            for (have = n0; have > 1; have = (have + 15) / 16) {       // (three times at most)
                const bool mine = 16 * tid < have;
                if (mine) {
                    double v1[16], v2[16];
#pragma unroll
                    for (int j = 0; j < 16; ++j) { v1[j] = s_sum[0][min(16 * tid + j, have - 1)]; v2[j] = s_sum[1][min(16 * tid + j, have - 1)]; }
                    s1 = v1[0]; s2 = v2[0];
#pragma unroll
                    for (int j = 1; j < 16; ++j)
                        if (16 * tid + j < have) { s1 += v1[j]; s2 += v2[j]; }
                }
                __syncthreads();
                if (mine) { s_sum[0][tid] = s1; s_sum[1][tid] = s2; }
                __syncthreads();
            }
            if (tid == 0) {
                float step, inv_step;
                step_pair_from_sums(s_sum[0][0], s_sum[1][0], q.n, q.s, step, inv_step);
                s_pair[0] = step; s_pair[1] = inv_step;
            }
            __syncthreads();
            inv = s_pair[1];
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (i % 8 == 0 && NT * i >= q.n) break;
            const int e = tid + NT * i;
            if (e >= q.n) continue;
            const float u = dither_u(q.idx_base + (uint64_t)e, q.k0, q.k1);
            const float kf = __builtin_floorf(__builtin_fmaf(x[i], inv, u)), kc = __builtin_amdgcn_fmed3f(kf, -127.0f, 127.0f);
            int k = (int)kc;
            if (kf != kc) {                                          // saturated, or not a number: code 0
                const bool nan = kf != kf;
                if (nan) k = 0;
                nonfinite += x[i] != x[i] || fabsf(x[i]) == __builtin_inff();
                sat += !nan && fabsf(kf) > 127.0f;
            }
            s_codes[e] = (int8_t)k;
            nnz += k != 0;
            top = max(top, (uint32_t)(k < 0 ? -k : k));
        }
        __syncthreads();
    };
    if (!writer) {
        const int block = (int)blockIdx.x - 1;
        const bool second = block >= a.first1;
        const FcdProblem &p = a.prob[second ? 1 : 0];
        fcd_form_tile(p, block - (second ? a.first1 : 0), fcd_lds, s_codes, quantise, [&] { return LAYER ? s_pair[0] : q.step; });
        return;
    }
    quantise();
    for (int e = tid; e < q.n; e += NT) q.codes[e] = s_codes[e];
    const float step = LAYER ? s_pair[0] : q.step;
    if constexpr (LAYER) {
        if (tid == 0) { q.step_out[0] = s_pair[0]; q.step_out[1] = s_pair[1]; }
        if (q.bias_grad) {
            // A column's codes are shared between `parts` threads, sixteen each at most: a thread a column took 27 us of
            // 4096x64x2 (the call: 54.1 us, now 19.5; with launches of their own 27.7).
            int *sums = (int *)s_v;                                  // (a place for every column: cols <= n; the gradients in it have been read)
            const int parts = max(NT / q.cols, 1), step_e = parts * q.cols;
            for (int c = tid; c < q.cols; c += NT) sums[c] = 0;
            __syncthreads();
            for (int e0 = tid; e0 < step_e; e0 += NT) {              // (once where columns share threads: step_e <= NT)
                int sum = 0;
                for (int e = e0; e < q.n; e += step_e) sum += s_codes[e];
                atomicAdd(&sums[e0 % q.cols], sum);
            }
            __syncthreads();
            for (int c = tid; c < q.cols; c += NT) q.bias_grad[c] = (float)((double)step * (double)sums[c]);
        }
    }
    if (q.stats) {
        __shared__ uint32_t s_stats[4][FCD_WAVES];
        nnz = wave_sum((int)nnz); sat = wave_sum((int)sat); nonfinite = wave_sum((int)nonfinite);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) top = max(top, (uint32_t)__shfl_xor((int)top, off));
        if ((tid & 63) == 0) { s_stats[0][tid >> 6] = nnz; s_stats[1][tid >> 6] = sat; s_stats[2][tid >> 6] = nonfinite; s_stats[3][tid >> 6] = top; }
        __syncthreads();
        if (tid == 0) {
            nnz = sat = nonfinite = top = 0;
            for (int w = 0; w < FCD_WAVES; ++w) { nnz += s_stats[0][w]; sat += s_stats[1][w]; nonfinite += s_stats[2][w]; top = max(top, s_stats[3][w]); }
            q.stats->nnz = nnz; q.stats->n_saturated = sat; q.stats->n_nonfinite = nonfinite; q.stats->max_abs_code = (int32_t)top; q.stats->reserved = 0;
        }
    }
}

hipError_t launch_fc_fused(const FcdArgs &a, const FusedQuant &q, int grid, size_t lds, hipStream_t s)
{
    static bool raised[2] = {false, false};                          // with its static LDS above 64 KiB: allowed per kernel, once
    const bool layer = q.s > 0.0f;
    void (*kernel)(FcdArgs, FusedQuant) = layer ? &fc_fused_kernel<true> : &fc_fused_kernel<false>;
    if (!raised[layer]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 64 << 10);
        if (e != hipSuccess) return e;
        raised[layer] = true;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * FCD_WAVES), lds, s, a, q);
    return hipGetLastError();
}

}  // namespace dbp
