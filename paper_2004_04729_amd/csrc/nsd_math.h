// Dither and step size of the quantiser, for the kernels of nsd.hip and for fc_fused_kernel.
#pragma once
#include "side_jobs.h"

namespace dbp {

namespace {

constexpr uint32_t kG = 0x9E3779B9u, kA = 0x6A09E667u, kC = 0xBB67AE85u;

__host__ __device__ inline uint32_t mix32(uint32_t x)
{
    x ^= x >> 16; x *= kA; x ^= x >> 15; x *= kC; x ^= x >> 16;
    return x;
}

// One 32-bit hash word per PAIR of elements; `k1c` already contains k1 + hi32(counter)*C.
__device__ __forceinline__ uint32_t hash_word(uint32_t counter_lo, uint32_t k0, uint32_t k1c)
{
    uint32_t h = (counter_lo ^ k0) * kG;
    h ^= h >> 16;
    h = (h + k1c) * kA;
    h ^= h >> 15;
    h *= kC;
    h ^= h >> 16;
    return h;
}

// u = (2m+1) * 2^-17 for a 16-bit m: build 1 + m*2^-16 in the mantissa, subtract (1 - 2^-17). Exact.
__device__ __forceinline__ float dither_from_m16(uint32_t m)
{
    return __uint_as_float(0x3F800000u | (m << 7)) - 0x1.ffffp-1f;
}

__device__ __forceinline__ float dither_u(uint64_t g, uint32_t k0, uint32_t k1)
{
    uint64_t c = g >> 1;
    uint32_t h = hash_word((uint32_t)c, k0, k1 + (uint32_t)(c >> 32) * kC);
    return dither_from_m16((g & 1) ? (h >> 16) : (h & 0xFFFFu));
}

// {Delta, 1/Delta} of Algorithm 1 from the sums of the values and of their squares: Delta = s * sqrt(S2/n - (S1/n)^2) in
// fp64, rounded to fp32 once.  A degenerate tensor (constant or non-finite gradient) gives {0, 0}: everything quantises
// to zero codes and the products are zero.
__device__ __forceinline__ void step_pair_from_sums(double S1, double S2, int64_t n, float s, float &step_out, float &inv_out)
{
    double var = n > 0 ? (S2 - S1 * S1 / (double)n) / (double)n : 0.0;
    if (var < 0.0) var = 0.0;
    const double sigma = __builtin_sqrt(var);
    const float step = (float)((double)s * sigma);
    const float inv = __fdiv_rn(1.0f, step);
    const bool ok = step > 0.0f && step < __builtin_inff() && inv >= 1.17549435e-38f && inv < __builtin_inff();
    step_out = ok ? step : 0.0f;
    inv_out = ok ? inv : 0.0f;
}

}  // namespace

}  // namespace dbp
