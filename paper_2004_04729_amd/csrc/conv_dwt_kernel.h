// Weight-gradient product of a 2-D convolution from int8 codes, Eq. (qdw) "analogously for convolutional layers", for any kernel
// size, stride, padding and plane size (internal header):
//   dW[k][c][r][s] = Delta * sum_{n,p,q} code[n][k][p][q] * X[n][c][p*st + r - pad][q*st + s - pad]
// fp32 activations as PL exact bf16 planes (three; two on request), int8 activations on int8 matrix cores with exact int32 sums.
//
// The reduction runs over pixels.  What makes that awkward on matrix cores is that a fragment wants 8 (16) consecutive reduction
// indices of one channel in a lane while a tap, a stride or a ragged row moves the activations by single pixels.  gfx950 reads LDS
// TRANSPOSED (ds_read_tr): sixteen lanes fetch rows of four (eight) pixels x sixteen channels and each keeps the pixels of one channel.  So:
//   * activations lie in LDS as [pixel][plane][32 channels], split into planes once when they are staged; the halo and everything
//     outside the image is zero.  A pixel is a row, so any tap of any output pixel is that pixel's row plus a constant: the lane
//     looks up its pixel's row once per step (a table, built once) and every tap adds a uniform offset.
//   * codes lie in LDS as bytes, a run of 8 (16) consecutive codes of a channel's plane a cell, cut and zero-filled once when they
//     are staged: a lane's fragment is one cell, for all taps and planes of the step.  (Read straight from memory, a fragment touches a
//     cache line per lane, again for every wavefront of other taps: 5x5 56x56 64->64 191 us against 86.)
//   * a wavefront owns 32*MF output channels x 32 input channels x G taps in registers (one tap: x G blocks of input channels); the
//     wavefronts of a workgroup divide output channels (kg), input channels (cb), taps (tg) and, where those are few, the steps (ps,
//     added up through LDS at the end).
//   * one tap with a stride reads every st-th pixel of every st-th row: only those are staged (1x1/2 512->1024 14x14 N=64: product 54 -> 43 us, with
//     int8 activations 51 -> 34; the column matrix 43 and 36).
//   * a unit is a band of output rows (or columns) of an image, or several small images; units go round the workgroups of a
//     tile, LDS is double buffered: the next unit's operands are loaded before this unit's steps and written after them.
//     Elements past a ragged band have zero codes and read the band's last pixels, not what lies behind them: a non-finite
//     activation reaches the taps that pair with it and no other.
// Partial sums of the workgroups that share a tile are added in a fixed order by conv_dwt_reduce_kernel.
// What bounds it: about 20 us of ends (launch, first loads from HBM, folding and writing partial sums); beyond them 60 % of the bf16 rate that
// matrix cores reach here.  Measured, kernel and reduction (us), against what served before: 128->256 28x28/2 N=64 50 / 67 (column matrix and
// fully connected kernels), 64->64 56x56 5x5 N=32 98 / 545 (generic kernel), 64->256 56x56 1x1 N=32 39 / 92 (batched 1x1 form).
#pragma once
#include "gemm_core.h"
#include "fc_kernel.h"

namespace dbp {

constexpr int DWT_MAX_LDS = 156 * 1024;
constexpr int DWT_RUN(bool i8) { return i8 ? 16 : 8; }

// What a wavefront owns: MF blocks of 32 output channels x 32 input channels x G taps or, with one tap (ONE), MF x G blocks of 32 channels;
// WAVES: the most wavefronts of a workgroup; ITEMS: staging items of a wavefront (64 pixels x 4 channels each); CREGS: registers
// of codes a thread stages.
template <int G, bool ONE> struct DwtShape;
template <> struct DwtShape<2, true>  { static constexpr int MF = 4, WAVES = 8,  ITEMS = 6, CREGS = 16; };
template <> struct DwtShape<4, true>  { static constexpr int MF = 2, WAVES = 8,  ITEMS = 6, CREGS = 16; };
template <> struct DwtShape<3, false> { static constexpr int MF = 2, WAVES = 12, ITEMS = 4, CREGS = 8; };
template <> struct DwtShape<4, false> { static constexpr int MF = 2, WAVES = 8,  ITEMS = 4, CREGS = 12; };

// Keeps a uniform counter of an unrolled loop a counter: the values of all rounds, hoisted out of the unit loop, overflow the scalar registers.
#define DWT_STEP(x) asm volatile("" : "+s"(x))

struct ConvDwtArgs {
    const int8_t *codes;          // [N][Kt][P][Q]
    const void   *X;              // [N][Ct][H][Wd]
    void *dW, *partial;           // [K][C][R][S]; partial: see conv_dwt_kernel's epilogue
    int N, C, H, Wd, K, S, T, st, pad, P, Q, Ct, Kt;    // T = R*S
    int st_load, st_lds;                                // st as the step between LDS pixels in the image (one tap reads no others) or between outputs in LDS
    int PB, bands, QB, cbands, NI;                      // output rows / columns per unit, bands of them, images per unit
    int units, units_per_split, n_split;
    int frame_w, frame, chunks;                         // LDS pixels per row and per image of a unit; chunks of 64 of the unit's
    int runs_row, runs_img, steps;                      // runs per row (flat bands: per band), per image; steps of two runs per unit
    int flat;                                           // whole rows: runs go on across row ends
    int last_rows, last_cols;                           // rows and columns of the last bands
    int tables, table_row, table_col;                   // tables of pixels; where those of the last bands begin (0: as large as the others)
    int kg, cb, ps, tg;                                 // wavefronts along output channels, input channels, steps, taps
    int tiles_k, tiles_c, tap_blocks;
    int blocks;                                         // blocks of 32 input channels a workgroup stages
    int x_bytes, buf_bytes;                             // activations of one LDS buffer, the buffer with its codes
    int tiny;                                           // planes shorter than a run
    int code_step;                                      // channels a pass of the code staging takes
    Scale scale;
    Gate gate;
};

typedef short    dwt_s4 __attribute__((ext_vector_type(4)));
typedef int      dwt_i2 __attribute__((ext_vector_type(2)));
typedef uint64_t dwt_u64 __attribute__((aligned(1)));

template <bool I8, int PL> __host__ __device__ constexpr int dwt_pitch() { return (I8 ? 32 : 64 * PL) + 8; }   // bytes per pixel: + 8 spreads the staging writes over the banks

__device__ __forceinline__ uint2 dwt_read_tr(const unsigned char *p, bool i8)
{
    typedef __attribute__((address_space(3))) dwt_s4 *p16;
    typedef __attribute__((address_space(3))) dwt_i2 *p8;
    if (i8) return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((p8)(p)));
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((p16)(p)));
}

// RAGGED: last bands smaller than the others, with a table of pixels of their own.  Choosing the table per unit costs 3 to 5 % in the loop (3x3/2
// 128->256 28x28 N=64 50 / 52 us), so whole bands and int8 operands (no NaN) have a form without.
template <bool I8, int PL, int G, bool ONE, bool RAGGED>
__global__ __launch_bounds__((64 * DwtShape<G, ONE>::WAVES), 1) void conv_dwt_kernel(ConvDwtArgs a)
{
    if (a.gate.closed()) return;
    using Acc = typename std::conditional<I8, i32x16, f32x16>::type;
    using Shape = DwtShape<G, ONE>;
    constexpr int MF = Shape::MF, MODE = I8 ? MODE_I8 : MODE_BF16, RUN = DWT_RUN(I8), PITCH = dwt_pitch<I8, PL>();
    constexpr int ITEMS = Shape::ITEMS, AD = RUN / 4, CITEMS = Shape::CREGS / AD;
    extern __shared__ uint4 dwt_lds[];
    unsigned char *lds = (unsigned char *)dwt_lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = (int)blockDim.x >> 6, threads = (int)blockDim.x;
    const int half = lane >> 5;

    // ---- which tile, which split, which part of it is this wavefront's
    int b = blockIdx.x;
    const int tiles = a.tiles_k * a.tiles_c * a.tap_blocks;
    const int split = b / tiles; b -= split * tiles;
    const int tb = b % a.tap_blocks; b /= a.tap_blocks;
    const int tile_k = b % a.tiles_k, tile_c = b / a.tiles_k;
    int w = wave;
    const int w_tg = w % a.tg; w /= a.tg;
    const int w_cb = w % a.cb; w /= a.cb;
    const int w_kg = w % a.kg, w_ps = w / a.kg;
    const int k_tile = tile_k * a.kg * 32 * MF, k0 = k_tile + w_kg * 32 * MF;
    const int c_tile = tile_c * a.blocks * 32;                                 // first input channel of the workgroup
    const int PQ = a.P * a.Q, HW = a.H * a.Wd;
    int tap_off[G];                                                       // taps past the last repeat it (their sums are not stored)
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int t = ONE ? 0 : min((tb * a.tg + w_tg) * G + g, a.T - 1), r = t / a.S;
        tap_off[g] = ONE ? g * (a.chunks * 64 * PITCH) : (r * a.frame_w + t - r * a.S) * PITCH;
    }

    // ---- a table, built once: run elements of a unit -> byte offset in LDS of the pixel that tap (0,0) reads
    uint32_t *t_pix = (uint32_t *)(lds + 2 * a.buf_bytes);
    // (and one each for the units of a ragged last row band, column band, and both)
    for (int table = 0, n = 2 * a.steps * RUN; table < (RAGGED ? a.tables : 1); ++table) {
        const int rows = a.table_row && (table & 1) ? a.last_rows : a.PB, cols = a.table_col && table * n >= a.table_col ? a.last_cols : a.QB;
        for (int e = tid; e < n; e += threads) {
            const int run = e / RUN, img = min(run / a.runs_img, a.NI - 1), f = run - run / a.runs_img * a.runs_img;
            int row = f / a.runs_row, col = (f - row * a.runs_row) * RUN + (e - run * RUN);
            if (a.flat) { row = col / a.Q; col -= row * a.Q; }
            row = min(row, rows - 1); col = min(col, cols - 1);            // elements past the band: its last pixels, their codes are zero
            t_pix[table * n + e] = (uint32_t)((img * a.frame + row * a.st_lds * a.frame_w + col * a.st_lds) * PITCH);
        }
    }
    for (int i = tid; i < 2 * a.buf_bytes / 16; i += threads) dwt_lds[i] = uint4{0u, 0u, 0u, 0u};   // nothing unset is ever multiplied
    // ---- staging: a wavefront keeps to one chunk of 64 pixels, a lane to its pixel, and takes every per_chunk-th quad of channels
    const int per_chunk = waves / a.chunks, my_chunk = wave / per_chunk, my_quad = wave - my_chunk * per_chunk;
    const bool stager = my_chunk < a.chunks;
    const int px = my_chunk * 64 + lane;
    int px_off, px_h, px_w, px_img;                                        // where the pixel comes from, relative to the unit's origin
    {
        px_img = px / a.frame;
        const int f = px - px_img * a.frame;
        px_h = f / a.frame_w; px_w = f - px_h * a.frame_w;
        px_h *= a.st_load; px_w *= a.st_load;
        px_off = px_img * a.Ct * HW + px_h * a.Wd + px_w;
        if (px_img >= a.NI) px_img = 1 << 24;                              // a pixel of no image
    }
    __syncthreads();

    // ---- units go round: (image group, row band, column band), columns fastest
    struct Unit { int n0, p0, q0; };
    auto unit_of = [&](int u) {
        Unit r;
        const int qb = u % a.cbands; u /= a.cbands;
        const int pb = u % a.bands; u /= a.bands;
        r.n0 = u * a.NI; r.p0 = pb * a.PB; r.q0 = qb * a.QB;
        return r;
    };
    auto advance = [&](Unit &r) {                                          // (no division: a wavefront has few instructions to spare)
        r.q0 += a.QB;
        if (r.q0 >= a.Q) { r.q0 = 0; r.p0 += a.PB; if (r.p0 >= a.P) { r.p0 = 0; r.n0 += a.NI; } }
    };

    const int64_t plane_bytes = (int64_t)HW * (I8 ? 1 : 4), skip_bytes = (int64_t)4 * (per_chunk - 1) * plane_bytes;
    uint32_t raw[ITEMS][4];
    auto fetch = [&](const Unit &u) {
        const int h0 = u.p0 * a.st - a.pad, w0 = u.q0 * a.st - a.pad;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[i][j] = 0u;
        const bool ok = stager && px_img < a.N - u.n0 && (uint32_t)(h0 + px_h) < (uint32_t)a.H && (uint32_t)(w0 + px_w) < (uint32_t)a.Wd;
        if (ok) {
            const char *at = (const char *)a.X + ((int64_t)u.n0 * a.Ct * HW + (int64_t)h0 * a.Wd + w0 + (int64_t)(c_tile + 4 * my_quad) * HW) * (I8 ? 1 : 4);   // uniform
            const uint32_t off = (uint32_t)px_off * (I8 ? 1u : 4u);
            int left = min(32 * a.blocks, a.C - c_tile) - 4 * my_quad;     // channels from this one on
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (left > j) {
                        if constexpr (I8) raw[i][j] = *(const uint8_t *)(at + off);
                        else raw[i][j] = *(const uint32_t *)(at + off);
                    }
                    at += plane_bytes;
                    DWT_STEP(at);
                }
                at += skip_bytes; left -= 4 * per_chunk;
                DWT_STEP(left);
            }
        }
    };
    auto stage = [&](unsigned char *buf) {
#pragma unroll
        for (int i = 0, quad = my_quad; i < ITEMS; ++i, quad += per_chunk) {
            DWT_STEP(quad);
            if (!stager || quad >= 8 * a.blocks) continue;                     // uniform
            unsigned char *dst = buf + (quad >> 3) * (a.chunks * 64 * PITCH) + px * PITCH + (quad & 7) * (I8 ? 4 : 8);
            if constexpr (I8) {
                *(uint32_t *)dst = raw[i][0] | (raw[i][1] << 8) | (raw[i][2] << 16) | (raw[i][3] << 24);
            } else if constexpr (PL == 3) {
                uint32_t h[4], m[4], l[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) split3_upper(__uint_as_float(raw[i][j]), h[j], m[j], l[j]);
                *(uint2 *)dst = uint2{upper_halves(l[1], l[0]), upper_halves(l[3], l[2])};
                *(uint2 *)(dst + 64) = uint2{upper_halves(m[1], m[0]), upper_halves(m[3], m[2])};
                *(uint2 *)(dst + 128) = uint2{upper_halves(h[1], h[0]), upper_halves(h[3], h[2])};
            } else {
                uint32_t h[2], l[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) split2_pk(__uint_as_float(raw[i][2 * j]), __uint_as_float(raw[i][2 * j + 1]), h[j], l[j]);
                *(uint2 *)dst = uint2{l[0], l[1]};
                *(uint2 *)(dst + 64) = uint2{h[0], h[1]};
            }
        }
    };

    Acc acc[MF][G];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][g][v] = 0;

    // ---- codes: a thread keeps to one run of the unit and takes that run of every code_step-th output channel of the tile
    const int n_runs = 2 * a.steps, KT = 32 * MF * a.kg, CPITCH = (n_runs + 1) * RUN;      // odd in runs: a fragment read spreads over the banks
    const int my_run = tid % n_runs, my_ch = tid / n_runs;
    const bool coder = my_ch < a.code_step;
    int r_img, r_row, r_col, r_off;
    {
        r_img = my_run / a.runs_img;
        const int f = my_run - r_img * a.runs_img;
        r_row = f / a.runs_row; r_col = (f - r_row * a.runs_row) * RUN;   // (flat bands: row 0, the column counts on)
        r_off = r_img * a.Kt * PQ + r_row * a.Q + r_col;
    }
    uint32_t craw[CITEMS][AD];
    int c_shift = 0, c_valid = 0;                                          // a run's loads are kept inside its plane, c_shift codes early; c_valid codes count
    auto fetch_codes = [&](const Unit &u) {
        const int rows = min(a.PB, a.P - u.p0), cols = min(a.QB, a.Q - u.q0);
        const int have = a.flat ? rows * a.Q - r_col : r_row < rows ? cols - r_col : 0;
        c_valid = r_img < a.NI && r_img < a.N - u.n0 ? min(max(have, 0), RUN) : 0;
        const int start = (u.p0 + r_row) * a.Q + u.q0 + r_col;
        c_shift = a.tiny ? 0 : max(start - (PQ - RUN), 0);
        if (coder && c_valid > 0) {
            const int8_t *base = a.codes + (int64_t)u.n0 * a.Kt * PQ;      // uniform
            const uint32_t o = (uint32_t)(r_off + u.p0 * a.Q + u.q0 - c_shift);
#pragma unroll
            for (int i = 0, k = 0; i < CITEMS; ++i, k += a.code_step) {
                DWT_STEP(k);
                if (k >= KT) break;                                        // uniform
                const int8_t *at = base + (o + (uint32_t)min(k_tile + my_ch + k, a.K - 1) * (uint32_t)PQ);
                if (a.tiny) {                                              // uniform: planes shorter than a run, code by code
#pragma unroll
                    for (int d = 0; d < AD; ++d) craw[i][d] = 0u;
#pragma unroll
                    for (int d = 0; d < RUN; ++d)
                        if (d < c_valid) craw[i][d / 4] |= (uint32_t)(uint8_t)at[d] << (8 * (d % 4));
                } else if constexpr (I8) {
                    const u32x4 v = *(const u32x4_unaligned *)at;
#pragma unroll
                    for (int d = 0; d < 4; ++d) craw[i][d] = v[d];
                } else {
                    const uint64_t v = *(const dwt_u64 *)at;
                    craw[i][0] = (uint32_t)v; craw[i][1] = (uint32_t)(v >> 32);
                }
            }
        }
    };
    // drop `shift` codes at the front of a run, keep `valid`
    auto cut_run = [&](uint32_t (&d)[AD], int shift, int valid) {
        if constexpr (I8) {
            const uint64_t lo = d[0] | (uint64_t)d[1] << 32, hi = d[2] | (uint64_t)d[3] << 32;
            const int s = 8 * min(shift, 16), v = 8 * valid;
            uint64_t l2 = s == 0 ? lo : s < 64 ? (lo >> s) | (hi << (64 - s)) : s < 128 ? hi >> (s - 64) : 0ull;
            uint64_t h2 = s < 64 ? hi >> s : 0ull;
            l2 &= v >= 64 ? ~0ull : (1ull << v) - 1;
            h2 &= v >= 128 ? ~0ull : v > 64 ? (1ull << (v - 64)) - 1 : 0ull;
            d[0] = (uint32_t)l2; d[1] = (uint32_t)(l2 >> 32); d[2] = (uint32_t)h2; d[3] = (uint32_t)(h2 >> 32);
        } else {
            uint64_t x = d[0] | (uint64_t)d[1] << 32;
            x = shift < 8 ? x >> (8 * shift) : 0ull;
            x &= valid >= 8 ? ~0ull : (1ull << (8 * valid)) - 1;
            d[0] = (uint32_t)x; d[1] = (uint32_t)(x >> 32);
        }
    };
    auto code_fragment = [&](const uint32_t (&d)[AD]) {
        if constexpr (I8) return u32x4{d[0], d[1], d[2], d[3]};
        else return u32x4{bf16x2_from_codes((int8_t)d[0], (int8_t)(d[0] >> 8)), bf16x2_from_codes((int8_t)(d[0] >> 16), (int8_t)(d[0] >> 24)),
                          bf16x2_from_codes((int8_t)d[1], (int8_t)(d[1] >> 8)), bf16x2_from_codes((int8_t)(d[1] >> 16), (int8_t)(d[1] >> 24))};
    };

    auto stage_codes = [&](unsigned char *buf) {
        unsigned char *dst = buf + a.x_bytes + my_ch * CPITCH + my_run * RUN;
        const bool cut = __any(c_valid < RUN || c_shift > 0);
#pragma unroll
        for (int i = 0, k = 0; i < CITEMS; ++i, k += a.code_step) {
            DWT_STEP(k);
            if (k >= KT) break;                                            // uniform
            if (cut) cut_run(craw[i], c_shift, c_valid);
            if (coder && my_ch + k < KT) {
                if constexpr (I8) *(u32x4 *)(dst + k * CPITCH) = u32x4{craw[i][0], craw[i][1], craw[i][2], craw[i][3]};
                else *(uint2 *)(dst + k * CPITCH) = uint2{craw[i][0], craw[i][1]};
            }
        }
    };

    // ---- steps of a unit: pixel rows of this lane in the transposed reads (two reads make a fragment)
    const int e_lane = I8 ? (lane & 15) >> 1 : (lane & 15) >> 2;            // which pixel of a read's four (eight) the lane fetches
    const int c_lane = I8 ? 16 * ((lane >> 4) & 1) + 8 * (lane & 1) : 2 * (16 * ((lane >> 4) & 1) + 4 * (lane & 3));   // byte of its channels
    const int x_base = w_cb * (ONE ? G : 1) * (a.chunks * 64 * PITCH) + c_lane, k_base = a.x_bytes + (w_kg * 32 * MF + (lane & 31)) * CPITCH;
    const int t_lane = half * RUN + e_lane;
    struct Head { uint32_t a[MF][AD], p0, p1; };                            // what a step starts from: its codes and its pixels
    auto head = [&](const unsigned char *buf, int table, int st) {
        Head h;
        const int run = 2 * min(st, a.steps - 1) + half, first = 2 * min(st, a.steps - 1) * RUN;                   // uniform
        const uint32_t *tp = t_pix + t_lane + (table + first);
        h.p0 = tp[0]; h.p1 = tp[RUN / 2];
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const unsigned char *at = buf + k_base + 32 * i * CPITCH + run * RUN;
            if constexpr (I8) {
                const u32x4 v = *(const u32x4 *)at;
#pragma unroll
                for (int d = 0; d < 4; ++d) h.a[i][d] = v[d];
            } else {
                const uint2 v = *(const uint2 *)at;
                h.a[i][0] = v.x; h.a[i][1] = v.y;
            }
        }
        return h;
    };
    auto multiply = [&](const unsigned char *buf, int table) {
        Head h = head(buf, table, w_ps);
        for (int st = w_ps; st < a.steps; st += a.ps) {
            const unsigned char *px0 = buf + x_base + h.p0, *px1 = buf + x_base + h.p1;
            u32x4 af[MF];
#pragma unroll
            for (int i = 0; i < MF; ++i) af[i] = code_fragment(h.a[i]);
            h = head(buf, table, st + a.ps);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                u32x4 bf[PL];
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) {
                    const uint2 lo = dwt_read_tr(px0 + tap_off[g] + 64 * pl, I8), hi = dwt_read_tr(px1 + tap_off[g] + 64 * pl, I8);
                    bf[pl] = u32x4{lo.x, lo.y, hi.x, hi.y};
                }
#pragma unroll
                for (int pl = 0; pl < PL; ++pl)
#pragma unroll
                    for (int i = 0; i < MF; ++i) Mma<MODE>::run(af[i], bf[pl], acc[i][g]);
            }
        }
    };

    const int u_begin = split * a.units_per_split, u_end = min(a.units, u_begin + a.units_per_split);
    Unit cur = unit_of(u_begin), next = cur;
    auto table_of = [&](const Unit &r) { return (r.p0 + a.PB >= a.P ? a.table_row : 0) + (r.q0 + a.QB >= a.Q ? a.table_col : 0); };
    int table = RAGGED ? table_of(cur) : 0;
    if (u_begin + 1 < u_end) advance(next);
    fetch(cur); fetch_codes(cur);
    stage(lds); stage_codes(lds);
    fetch(next); fetch_codes(next);
    __syncthreads();
    for (int u = u_begin; u < u_end; ++u) {
        const int ib = (u - u_begin) & 1;
        multiply(lds + ib * a.buf_bytes, table);
        stage(lds + (1 - ib) * a.buf_bytes); stage_codes(lds + (1 - ib) * a.buf_bytes);
        if constexpr (RAGGED) table = table_of(next);
        if (u + 2 < u_end) advance(next);
        fetch(next); fetch_codes(next);
        __syncthreads();
    }

    // ---- the wavefronts that shared a tile's steps add up, in halves (a fixed order); the buffers are free by now
    using E = typename std::conditional<I8, int32_t, float>::type;
    const int tile_waves = a.tg * a.cb * a.kg, w_in_tile = wave % tile_waves;
    for (int h = a.ps >> 1; h > 0; h >>= 1) {
        uint32_t *slot = (uint32_t *)lds + ((w_ps % h) * tile_waves + w_in_tile) * (MF * G * 16 * 64) + lane;
        if (w_ps >= h && w_ps < 2 * h) {
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int v = 0; v < 16; ++v) slot[((i * G + g) * 16 + v) * 64] = __builtin_bit_cast(uint32_t, (E)acc[i][g][v]);
        }
        __syncthreads();
        if (w_ps < h) {
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][g][v] += __builtin_bit_cast(E, slot[((i * G + g) * 16 + v) * 64]);
        }
        __syncthreads();
    }
    if (w_ps != 0) return;

    // ---- D[ii][lane & 31] of a block: output channel 32*i + ii, input channel lane & 31
    if (a.n_split > 1) {
        // partial[split][tile][wavefront][i][g][four v][lane][4]
        uint32_t *dst = (uint32_t *)a.partial + ((int64_t)blockIdx.x * tile_waves + w_in_tile) * (MF * G * 1024) + 4 * lane;
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    u32x4 t;
#pragma unroll
                    for (int v = 0; v < 4; ++v) t[v] = __builtin_bit_cast(uint32_t, (E)acc[i][g][4 * q + v]);
                    *(u32x4 *)(dst + ((i * G + g) * 4 + q) * 256) = t;
                }
        return;
    }
    const float sc = I8 ? 1.0f : a.scale.get();
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int t = ONE ? 0 : (tb * a.tg + w_tg) * G + g, c = c_tile + 32 * (ONE ? w_cb * G + g : w_cb) + (lane & 31);
        if (t >= a.T || c >= a.C) continue;
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = k0 + 32 * i + 8 * (v >> 2) + 4 * half + (v & 3);
                if (k >= a.K) continue;
                E *out = (E *)a.dW + ((int64_t)k * a.C + c) * a.T + t;
                if constexpr (I8) *out = acc[i][g][v]; else *out = sc * acc[i][g][v];
            }
    }
}

// Sum over the splits.  A workgroup takes 8 output channels (four v of both halves) x 32 input channels of a tile and `tch` taps:
// the partials are read in whole lines by ZG groups of threads (a share of the splits each, in order, the shares added in
// order), go through LDS and leave as stretches of `tch` outputs per input channel.
template <int G, bool ONE>
__global__ __launch_bounds__(1024) void conv_dwt_reduce_kernel(ConvDwtArgs a, int i8, int tch, int tap_chunks, int ZG)
{
    if (a.gate.closed()) return;
    constexpr int MF = DwtShape<G, ONE>::MF;
    extern __shared__ uint32_t dwt_red[];
    int b = blockIdx.x;
    const int t0 = (b % tap_chunks) * tch; b /= tap_chunks;
    const int q = b % 4; b /= 4;
    const int i = b % MF; b /= MF;
    const int blk = b % a.blocks; b /= a.blocks;
    const int w_cb = ONE ? blk / G : blk, g_one = ONE ? blk - w_cb * G : 0;
    const int w_kg = b % a.kg; b /= a.kg;
    const int tile_k = b % a.tiles_k, tile_c = b / a.tiles_k;
    const int k0 = ((tile_k * a.kg + w_kg) * MF + i) * 32 + 8 * q, c0 = (tile_c * a.blocks + blk) * 32;
    const int tile_waves = a.tg * a.cb * a.kg, tiles = a.tiles_k * a.tiles_c * a.tap_blocks;
    const int64_t per_split = (int64_t)tiles * tile_waves * (MF * G * 1024);
    const int nt = min(tch, a.T - t0), items = 64 * nt;
    if (k0 >= a.K || c0 >= a.C) return;
    const int threads = (int)blockDim.x, per_z = (a.n_split + ZG - 1) / ZG;
    u32x4 *sums = (u32x4 *)dwt_red;                                         // [ZG][64 * tch]
    for (int x0 = threadIdx.x; x0 < ZG * 64 * tch; x0 += threads) {
        const int zg = x0 / (64 * tch), e = x0 - zg * (64 * tch);
        u32x4 r = {0u, 0u, 0u, 0u};
        if (e < items) {
            const int t = t0 + (e >> 6), lane = e & 63;
            const int slot = ONE ? 0 : t / G, g = ONE ? g_one : t - slot * G, tb = slot / a.tg, w_tg = slot - tb * a.tg;
            const int tile = (tile_c * a.tiles_k + tile_k) * a.tap_blocks + tb, w = (w_kg * a.cb + w_cb) * a.tg + w_tg;
            const uint32_t *src = (const uint32_t *)a.partial + ((int64_t)tile * tile_waves + w) * (MF * G * 1024) + ((i * G + g) * 4 + q) * 256 + 4 * lane;
            float s[4] = {0.f, 0.f, 0.f, 0.f};
            int32_t n[4] = {0, 0, 0, 0};
            const int z1 = min(a.n_split, (zg + 1) * per_z);
            for (int z = zg * per_z; z < z1; z += 8) {                      // eight loads in flight, sums in split order
                u32x4 x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = *(const u32x4 *)(src + (int64_t)min(z + j, z1 - 1) * per_split);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (z + j < z1) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) { s[v] += __uint_as_float(x[j][v]); n[v] += (int32_t)x[j][v]; }
                    }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) r[v] = i8 ? (uint32_t)n[v] : __float_as_uint(s[v]);
        }
        sums[x0] = r;
    }
    __syncthreads();
    const float sc = i8 ? 1.0f : a.scale.get();
    const int row = 32 * tch;
    for (int o = threadIdx.x; o < 8 * row; o += threads) {
        const int r = o / row, c = (o - r * row) / tch, t = o - r * row - c * tch;
        if (k0 + r >= a.K || c0 + c >= a.C || t >= nt) continue;
        const uint32_t *src = dwt_red + 4 * (64 * t + 32 * (r >> 2) + c) + (r & 3);
        float s = 0.f;
        int32_t n = 0;
        for (int zg = 0; zg < ZG; ++zg) { const uint32_t x = src[zg * (64 * tch) * 4]; s += __uint_as_float(x); n += (int32_t)x; }
        ((uint32_t *)a.dW)[((int64_t)(k0 + r) * a.C + c0 + c) * a.T + t0 + t] = i8 ? (uint32_t)n : __float_as_uint(sc * s);
    }
}

}  // namespace dbp
