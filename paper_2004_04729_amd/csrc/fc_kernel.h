// The two fully connected products, Eqs. (qda)/(qdw), as the kernels of fc2_kernel.h, fc2_i8_kernel.h and
// fc_direct_kernel.h see them (internal header).
//
//   dX[b,i] = Delta * sum_o code[b,o] W[o,i]      A = codes, reduction index contiguous  (a_kfast)
//   dW[o,i] = Delta * sum_b code[b,o] X[b,i]      A = codes^T, reduction index strided    (!a_kfast)
//
// In both products the dense operand is stored [reduction][column] with columns contiguous, so one B path serves both.
// ONE launch computes BOTH products: dX streams W from HBM and writes little, dW reads little and writes its whole output,
// so mixing the two keeps loads, matrix cores and stores busy at the same time instead of in chip-wide bursts.
// Split-K partials are summed in split order by a small second launch for both products (deterministic; summing in the last
// workgroup to arrive needs device-scope fences, and on this multi-XCD part each writes back a whole L2: 10x slower).
#pragma once
#include "gemm_core.h"

namespace dbp {

struct FcProblem {
    const int8_t *A; int64_t lda;     // a_kfast: A[m*lda + k]   else: A[k*lda + m]
    const float  *B; int64_t ldb;     // B[k*ldb + n]
    float *out; int64_t ldc;          // out[m*ldc + n]
    float *partial;                   // [tile][split][256*128] in thread order (n_split > 1)
    int M, N, K, k_per_split, n_split, tiles_m, n_items;
    Scale scale;
    int a_kfast;
    // Batched form of the kernel of fc2_kernel.h (both operands reduction-contiguous, one pair per image, accumulated):
    // A_img[m*lda + k], B_img[n*ldb + k], k < nt_pq; image i at A + i*nt_a_img, B + i*nt_b_img (elements); the
    // reduction axis K counts nt_spi windows of 32 per image.  nt_pq == 0: the plain form above.
    int nt_pq, nt_spi;
    int64_t nt_a_img, nt_b_img;
};
// gx > 0 (kernels of fc2_kernel.h / fc2_i8_kernel.h): the first gx workgroups of the launch take the items of problem 0, the
// others those of problem 1, each group dealing its items round robin; gx == 0: one list for both, dealt in a serpentine.
struct FcPairArgs { FcProblem prob[2]; StatsJob stats; int gx = 0; Gate gate; };

__device__ __forceinline__ uint32_t bf16x2_from_codes(int a, int b)
{
    // integers up to 127 in magnitude are exact in bf16 = the upper half of their fp32 image
    return __builtin_amdgcn_perm(__float_as_uint((float)b), __float_as_uint((float)a), 0x07060302u);
}

__device__ __forceinline__ uint32_t upper_halves(uint32_t hi_word, uint32_t lo_word)
{
    return __builtin_amdgcn_perm(hi_word, lo_word, 0x07060302u);    // {hi_word[31:16], lo_word[31:16]}
}

}  // namespace dbp
