// What the quantiser leaves to a later kernel of the stream (StatsJob): the sum of its statistics records and the bias
// gradient, done by workgroups that a launch adds for them (internal header).
#pragma once
#include "common.h"

namespace dbp {

// Bias gradient of channel `ch` by a workgroup of NT threads: Delta * (sum of the channel's codes over all images), one fp64
// product rounded to fp32; the sum is of integers, so its order does not matter.
__device__ __forceinline__ void bias_of_channel(const StatsJob &j, int ch, int NT)
{
    const double d = j.step_dev ? (double)j.step_dev[0] : (double)j.step;
    long long sum = 0;
    if (j.tile_sums) {
        // a stretch's sum sits at its last tile: the last of a row, of a wavefront's run, or of the tensor (which ends a row)
        const int64_t total = j.images * j.tiles_per_row;
        for (int64_t i = threadIdx.x; i < total; i += NT) {
            const int64_t img = i / j.tiles_per_row, seg = i - img * j.tiles_per_row;
            const int64_t t = (img * j.bias_len + ch) * j.tiles_per_row + seg;
            if (seg == j.tiles_per_row - 1 || (t + 1) % j.run == 0) sum += j.tile_sums[t];
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    } else {
        // 16-byte pieces of all the channel's planes in turn, four loads in flight: the codes come from memory, about 2 us a round
        // (a plane's last piece ends at its last code and gives up what it repeats; tiny planes go byte by byte)
        const int plane = (int)j.plane, bytes = plane < 16 ? 1 : 16;
        const int pieces = (plane + bytes - 1) / bytes, step_i = NT / pieces, step_w = NT % pieces;
        const int64_t img_bytes = j.bias_len * j.plane;
        const int8_t *base = j.bias_codes + ch * j.plane;
        int img = (int)threadIdx.x / pieces, w = (int)threadIdx.x - img * pieces, acc = 0;
        while (img < (int)j.images) {
            u32x4 v[4];
            int drop[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = img < (int)j.images;
                const int8_t *p = base + (in ? img : 0) * img_bytes;
                const int at = min(bytes * w, plane - bytes);
                drop[u] = in ? bytes * w - at : 16;
                if (bytes == 16) v[u] = *(const u32x4_unaligned *)(p + at);
                else v[u] = u32x4{(uint32_t)(uint8_t)p[at], 0u, 0u, 0u};
                img += step_i; w += step_w;
                if (w >= pieces) { w -= pieces; ++img; }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int gone = min(max(drop[u] - 4 * d, 0), 4);
                    const int x = gone == 4 ? 0 : (int)(v[u][d] >> (8 * gone));
                    acc += (x << 24 >> 24) + (x << 16 >> 24) + (x << 8 >> 24) + (x >> 24);
                }
        }
        sum = wave_sum(acc);                                           // (the caller keeps such channels below 2^31 / 127 codes)
    }
    __shared__ long long s_bias[16];
    if ((threadIdx.x & 63) == 0) s_bias[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long all = 0;
        for (int w = 0; w < NT / 64; ++w) all += s_bias[w];
        j.bias_grad[ch] = (float)(d * (double)all);
    }
}

// The statistics, by one workgroup of NT (at most 1024) threads.  All loads are in flight at once (the sums are of integers: any order
// gives the same result).
__device__ __forceinline__ void side_stats(const StatsJob &job, int NT)
{
    if (job.n > 0) {
        __shared__ uint64_t s_sum[3][16];
        __shared__ uint32_t s_max[16];
        uint64_t nnz = 0, sat = 0, nf = 0; uint32_t mx = 0;
        for (int base = 0; base < job.n; base += NT * 8) {
            u32x4 q[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int i = base + (int)threadIdx.x + NT * r;
                q[r] = i < job.n ? job.partials[i] : u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) { nnz += q[r].x; sat += q[r].y; nf += q[r].z; mx = max(mx, q[r].w); }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            nnz += __shfl_xor((unsigned long long)nnz, off); sat += __shfl_xor((unsigned long long)sat, off);
            nf += __shfl_xor((unsigned long long)nf, off); mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
        }
        const int w = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) { s_sum[0][w] = nnz; s_sum[1][w] = sat; s_sum[2][w] = nf; s_max[w] = mx; }
        __syncthreads();
        if (threadIdx.x == 0) {
            nnz = sat = nf = 0; mx = 0;
            for (int v = 0; v < NT / 64; ++v) { nnz += s_sum[0][v]; sat += s_sum[1][v]; nf += s_sum[2][v]; mx = max(mx, s_max[v]); }
            job.out->nnz = nnz; job.out->n_saturated = sat; job.out->n_nonfinite = nf;
            job.out->max_abs_code = (int32_t)mx; job.out->reserved = 0;
            write_density_flags(job, nnz);
        }
    }
}

// Workgroup `i` of job.workgroups(): the bias gradient first (from int64 sums a stretch of columns each: one workgroup for all of them is a chain of
// memory latencies, the call of 16x64x65536 81 us instead of 44), then the statistics.
__device__ __forceinline__ void side_job(const StatsJob &job, int i, int NT)
{
    if (i >= (int)job.bias_groups()) { side_stats(job, NT); return; }
    if (job.per_channel()) { bias_of_channel(job, i, NT); return; }
    const double d = job.step_dev ? (double)job.step_dev[0] : (double)job.step;
    const int64_t first = (int64_t)i * StatsJob::kBiasPerGroup, end = min(job.bias_len, first + StatsJob::kBiasPerGroup);
    for (int64_t c = first + threadIdx.x; c < end; c += NT) job.bias_grad[c] = (float)(d * (double)job.bias_sums[c]);
}

}  // namespace dbp
