// Input-gradient product of a convolution (see conv_dx_kernel.h for the problem, the prepared weights and the strided classes)
// for layers with few output pixels: the wavefronts of a workgroup divide the REDUCTION instead of channels and pixels.
//
//   * A workgroup owns 32 input channels x up to 32*NB pixels, a run of pixels of one image or several whole small images
//     (7x7 planes: 196 of 224 pixel columns in use, where a tile of one image used 49 of 64).  Every wavefront holds the whole
//     tile in registers, so a weight fragment (from L2, the scarcer stream) is used for NB pixel blocks.  conv_dx_kernel fills the
//     chip on such layers only with tiles of two blocks, and waits for weights: 3.7 times the L2 reads here.
//   * Wavefront w takes the pairs of k-groups (2*G output channels) w, w + waves, ...: it stages the codes of its own pair into
//     LDS of its own, as cells [k-group][patch pixel][G channels], and nobody else reads them.  No barrier before the end: the
//     wavefronts of a SIMD drift apart and one's staging runs beside the other's matrix instructions.  LDS operations of a
//     wavefront are executed in order, so one buffer is enough; the next pair's codes are on their way as global loads.
//   * At the end the wavefronts add up through LDS by recursive halving, in a fixed order: in every round a wavefront hands half of
//     its rows to its partner and keeps the other half, so that all of them store.
//   * A workgroup lives for a few pairs only, so its beginning counts: the first weights and codes are asked for before the indices of the LDS
//     cells are worked out, and these take no integer division (kernel, us: 14x14 49.0 -> 45.6, 7x7 48.2 -> 42.6).
// What bounds it: matrix instructions and their operands (256->256 14x14 N=64: matrix cores busy 56 % of the cycles in which a CU has a workgroup,
// 43 % of the launch; LDS bank conflicts 11 %), and that a CU has nothing to do for a quarter of so short a launch.  Every workgroup stages its
// pixels' codes for 32 channels only, so layers of many channels AND many pixels stay on conv_dx_kernel (conv_dx_workgroup_us).
// Measured, preparation and kernel (us), conv_dx_kernel (with 32x32x16 matrix instructions) / here: 256->256 14x14 N=64 65.6 / 48, 512->512 7x7 N=64 82.2 / 53,
// 16->537 8x8 N=119 69.7 / 22.0, 40->840 3x3/2 8x8 N=83 80.9 / 27.4, 332->37 5x5 16x16 N=52 63.9 / 49.0; 64->64 32x32 N=128 39.0 / 49.6.
#pragma once
#include "conv_dx_kernel.h"

namespace dbp {

// Patch-fill items (k-group, aligned dword of an image's codes) per lane and pair, at most: as many as leave the registers to the tile.  Small tiles
// take the rows of wide planes under large kernels too (5x5 on 88x88 planes, 48->264 N=12: no tile of conv_dx_kernel fits, the whole call 2087 us on the generic kernel, 717 here).
constexpr int cds_items(int nb) { return nb == 2 ? 6 : 3; }
constexpr int CDS_MAX_LDS = 156 * 1024;          // of a workgroup; two of four wavefronts share a CU where they fit

// T9: nine taps, the tap loop unrolled (exact wait counts: the codes' loads stay in flight behind the weights').
template <int NB, int MODE, bool STRIDED, bool T9>
__device__ __forceinline__ void conv_dx_split_body(const ConvDxArgs &a, int b)
{
    using TR = CdxTraits<MODE>;
    using Acc = typename TR::Acc;
    using E = typename TR::Out;
    constexpr int G = TR::G, PL = TR::PL;
    constexpr int NB0 = (NB + 1) / 2, NB1 = NB - NB0, ITEMS = cds_items(NB);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int waves = (int)blockDim.x >> 6;
    const int lcol = lane & 31, lhalf = lane >> 5;

    // ---- which tile: channel blocks fastest, so that an XCD (workgroups go round them) keeps to few channel blocks' weights
    const int cb = b % a.cgroups; b /= a.cgroups;
    const int tile = b % a.tiles, n0 = b / a.tiles * a.NI;
    const int ni = min(a.NI, a.N - n0);
    const int j0 = tile * 32 * NB;
    const int j_end = a.NI > 1 ? ni * a.PI : min(j0 + 32 * NB, a.PI);

    // patch geometry, the same for every image of the tile
    const int h_first = a.NI > 1 ? 0 : j0 / a.Wd, h_last = a.NI > 1 ? a.H - 1 : (j_end - 1) / a.Wd;
    const int p_lo = h_first + a.pad - (a.R - 1), q_lo = (STRIDED ? a.pad_w : a.pad) - (a.S - 1);
    const int p_a = max(p_lo, 0), p_b = min(h_last + a.pad, a.P - 1);
    const int kg_cells = a.patch_cells;                          // of one k-group: NI images
    uint4 *mine = cdx_lds + wave * a.wave_cells;                 // 2 * kg_cells and one that nobody reads

    // ---- weights: a step is a tap of a pair; a cursor walks the wavefront's steps ahead of them and stays on the last one
    const int RS = T9 ? 9 : a.R * a.S;
    const int64_t tap_stride = (int64_t)PL * a.Cp * a.KG;        // cells
    const uint32_t wl = (uint32_t)(lhalf * PL * a.Cp + cb * 32 + lcol);
    const int last_pair = wave + (a.pairs - 1 - wave) / waves * waves;           // (wave < pairs)
    int l_pair = wave, l_tap = 0;
    auto next_load = [&](u32x4 (&dst)[PL]) {
        const uint4 *row = a.wp + (l_tap * tap_stride + (int64_t)l_pair * (2 * PL) * a.Cp);     // uniform
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) { const uint4 t = row[wl + (uint32_t)(pl * a.Cp)]; dst[pl] = u32x4{t.x, t.y, t.z, t.w}; }
        if (++l_tap == RS) {
            if (l_pair < last_pair) { l_tap = 0; l_pair += waves; }
            else l_tap = RS - 1;
        }
    };
    u32x4 f0[PL], f1[PL], f2[PL];
    const bool active = wave < a.pairs;                          // uniform; (the plan leaves no wavefront without a pair)
    if (active) {
        next_load(f0);
        if constexpr (T9) next_load(f1);
    }

    // ---- patch-fill items of this lane; places outside the patch go to the cell that nobody reads
    const int f_a = (p_a * a.Q) & ~3;
    const int n_dw = p_b >= p_a ? ((p_b + 1) * a.Q - f_a + 3) >> 2 : 0;
    const int n_items = 2 * ni * n_dw;
    const float r_dw = cdx_rcp(n_dw), r_all = cdx_rcp(ni * n_dw), r_q = cdx_rcp(a.Q), r_w = cdx_rcp(a.Wd), r_pi = cdx_rcp(a.PI);
    uint32_t item_goff[ITEMS], item_cell[ITEMS][2];
    int item_k[ITEMS], item_cell0[ITEMS], item_rel[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int it = lane + 64 * i;
        item_goff[i] = 0u; item_k[i] = 0; item_cell0[i] = 0; item_rel[i] = -4;     // none: before the patch
        if (it < n_items) {
            const int kgl = cdx_div(it, r_all), rest = it - kgl * (ni * n_dw), im = cdx_div(rest, r_dw), f = rest - im * n_dw;
            item_k[i] = kgl * G;
            item_goff[i] = (uint32_t)(im * (int)a.code_img + f_a + 4 * f);
            item_cell0[i] = kgl * kg_cells + im * a.img_cells;
            item_rel[i] = f_a + 4 * f - p_a * a.Q;
        }
    }
    uint32_t raw[ITEMS][G];
    const int8_t *img = a.codes + (int64_t)n0 * a.code_img;
    // Channels past the last one repeat it: their weights are zero.
    auto fetch = [&](int pair) {
        const int8_t *src = img + (int64_t)pair * (2 * G) * a.PQ;                // uniform
        const int last = a.K - 1 - pair * 2 * G;                                  // uniform, >= 0
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (64 * i >= n_items) break;                                         // uniform
            uint32_t off = item_goff[i] + (uint32_t)(min(item_k[i], last) * a.PQ);
#pragma unroll
            for (int kq = 0; kq < G; ++kq) {
                raw[i][kq] = *(const uint32_t *)(src + off);
                off += item_k[i] + kq < last ? (uint32_t)a.PQ : 0u;
            }
        }
    };
    if (active) fetch(wave);
    for (int i = lane; i < a.wave_cells; i += 64) mine[i] = uint4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (64 * i >= n_items) break;                                             // uniform
        uint32_t cells[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int rel = item_rel[i] + e, p = p_a + cdx_div(rel, r_q), q = rel - (p - p_a) * a.Q;
            const bool need = rel >= 0 && p <= p_b && q >= q_lo && q - q_lo < a.pw;
            cells[e] = need ? (uint32_t)(item_cell0[i] + (p - p_lo) * a.pw + (q - q_lo)) : (uint32_t)(2 * kg_cells);
        }
        item_cell[i][0] = cells[0] | (cells[1] << 16);
        item_cell[i][1] = cells[2] | (cells[3] << 16);
    }
    auto store = [&]() {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (64 * i >= n_items) break;                                         // uniform
            if constexpr (MODE == MODE_I8) {
                uint32_t t[4][4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const uint32_t r0 = raw[i][4 * g], r1 = raw[i][4 * g + 1], r2 = raw[i][4 * g + 2], r3 = raw[i][4 * g + 3];
                    const uint32_t x0 = __builtin_amdgcn_perm(r1, r0, 0x05010400u), x1 = __builtin_amdgcn_perm(r3, r2, 0x05010400u);
                    const uint32_t y0 = __builtin_amdgcn_perm(r1, r0, 0x07030602u), y1 = __builtin_amdgcn_perm(r3, r2, 0x07030602u);
                    t[g][0] = __builtin_amdgcn_perm(x1, x0, 0x05040100u); t[g][1] = __builtin_amdgcn_perm(x1, x0, 0x07060302u);
                    t[g][2] = __builtin_amdgcn_perm(y1, y0, 0x05040100u); t[g][3] = __builtin_amdgcn_perm(y1, y0, 0x07060302u);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    mine[(item_cell[i][e >> 1] >> (16 * (e & 1))) & 0xFFFFu] = uint4{t[0][e], t[1][e], t[2][e], t[3][e]};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    mine[(item_cell[i][e >> 1] >> (16 * (e & 1))) & 0xFFFFu] =
                        uint4{cdx_bf16_pair(raw[i][0], raw[i][1], e), cdx_bf16_pair(raw[i][2], raw[i][3], e),
                              cdx_bf16_pair(raw[i][4], raw[i][5], e), cdx_bf16_pair(raw[i][6], raw[i][7], e)};
            }
        }
    };

    // ---- per-lane patch cell of each pixel, for the last tap; tap (r, s) adds (R-1-r)*pw + S-1-s
    int lane_cell[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        int j = min(j0 + 32 * nb + lcol, j_end - 1);            // tail lanes compute a valid pixel again; not stored
        const int im = a.NI > 1 ? cdx_div(j, r_pi) : 0;
        j -= im * a.PI + h_first * a.Wd;
        const int h = cdx_div(j, r_w), w = j - h * a.Wd;
        lane_cell[nb] = im * a.img_cells + h * a.pw + w + lhalf * kg_cells;
    }

    Acc acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[nb][v] = 0;

    // Code fragments in two groups of blocks: a group is read from LDS behind the other group's matrix instructions.
    u32x4 bA[NB0], bB[NB1];
    auto read_a = [&](int off) {
#pragma unroll
        for (int nb = 0; nb < NB0; ++nb) { const uint4 t = mine[lane_cell[nb] + off]; bA[nb] = u32x4{t.x, t.y, t.z, t.w}; }
    };
    auto read_b = [&](int off) {
#pragma unroll
        for (int nb = 0; nb < NB1; ++nb) { const uint4 t = mine[lane_cell[NB0 + nb] + off]; bB[nb] = u32x4{t.x, t.y, t.z, t.w}; }
    };
    auto step = [&](u32x4 (&nxt_w)[PL], const u32x4 (&cur)[PL], int off, int nxt) {
        next_load(nxt_w);
        read_b(off);
#pragma unroll
        for (int pl = 0; pl < PL; ++pl)
#pragma unroll
            for (int nb = 0; nb < NB0; ++nb) Mma<MODE>::run(cur[pl], bA[nb], acc[nb]);
        read_a(nxt);
#pragma unroll
        for (int pl = 0; pl < PL; ++pl)
#pragma unroll
            for (int nb = 0; nb < NB1; ++nb) Mma<MODE>::run(cur[pl], bB[nb], acc[NB0 + nb]);
    };

    if (active) {
        for (int pair = wave; pair < a.pairs; pair += waves) {
            // The lanes of a wavefront exchange codes through its LDS: in order for the hardware, fenced for the compiler.
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            store();
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            fetch(min(pair + waves, last_pair));                 // in flight during the matrix instructions (the last pair once more, unused)
            if constexpr (T9) {
                read_a(2 * a.pw + 2);
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const int o = (2 - r) * a.pw;
                    step(f2, f0, o + 2, o + 1);
                    step(f0, f1, o + 1, o);
                    step(f1, f2, o, r < 2 ? o - a.pw + 2 : o);   // (the last step reads its own codes again: the next ones are not there yet)
                }
            } else {
                int r = a.R - 1, s = a.S - 1, off = r * a.pw + s;
                read_a(off);
                for (int tap = 0; tap < RS; ++tap) {
                    if (--s < 0) { s = a.S - 1; --r; }
                    const int nxt = r < 0 ? off : r * a.pw + s;
                    step(f1, f0, off, nxt);
                    off = nxt;
#pragma unroll
                    for (int pl = 0; pl < PL; ++pl) f0[pl] = f1[pl];
                }
            }
        }
    }

    // ---- add up: lane holds pixel column lcol, channel rows 8*(v/4) + 4*lhalf + v%4 of its block; a round halves a wavefront's v
    uint32_t *fold = (uint32_t *)cdx_lds;
    int v_first = 0;
    auto halve = [&](auto vc, int h) {
        constexpr int V2 = decltype(vc)::value / 2;
        const bool upper = (wave & h) != 0;                      // uniform
        __syncthreads();
        constexpr int U = V2 < 4 ? V2 : 4;                       // elements an LDS access takes
        typedef uint32_t Piece __attribute__((ext_vector_type(U)));
        Piece *dst = (Piece *)fold + wave * (NB * V2 / U * 64) + lane;
        const Piece *src = (const Piece *)fold + (wave ^ h) * (NB * V2 / U * 64) + lane;
        auto give = [&](int first) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < V2; v += U) {
                    Piece t;
#pragma unroll
                    for (int u = 0; u < U; ++u) t[u] = __builtin_bit_cast(uint32_t, (E)acc[nb][first + v + u]);
                    dst[(nb * V2 + v) / U * 64] = t;
                }
        };
        if (upper) {
            give(0);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < V2; ++v) acc[nb][v] = acc[nb][V2 + v];
        } else {
            give(V2);
        }
        __syncthreads();
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < V2; v += U) {
                const Piece t = src[(nb * V2 + v) / U * 64];
#pragma unroll
                for (int u = 0; u < U; ++u) { const uint32_t x = t[u]; acc[nb][v + u] += __builtin_bit_cast(E, x); }
            }
        v_first += upper ? V2 : 0;
    };
    const bool eight = waves == 8;
    halve(std::integral_constant<int, 16>{}, waves >> 1);
    halve(std::integral_constant<int, 8>{}, waves >> 2);
    if (eight) halve(std::integral_constant<int, 4>{}, 1);

    // ---- store what this wavefront kept: v_first .. v_first + 4 (eight wavefronts: 2)
    E *out = (E *)a.dX + (int64_t)n0 * a.dx_img;                 // offsets inside a tile's images fit 31 bits (host check)
    const float sc = MODE == MODE_I8 ? 1.0f : a.scale.get();
    const int opi = STRIDED ? a.oPI : a.PI;
    const int c0 = cb * 32 + 8 * (v_first >> 2) + 4 * lhalf + (v_first & 3);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        int j = j0 + 32 * nb + lcol;
        if (j >= j_end) continue;
        const int im = a.NI > 1 ? cdx_div(j, r_pi) : 0;
        j -= im * a.PI;
        int px = j;
        if constexpr (STRIDED) { const int h = h_first + cdx_div(j - h_first * a.Wd, r_w), w = j - h * a.Wd; px = (a.ost * h + a.oh0) * a.oW + a.ost * w + a.ow0; }
        const int off = im * (int)a.dx_img + c0 * opi + px;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if ((v < 2 || !eight) && c0 + v < a.C) {
                if constexpr (MODE == MODE_I8) out[off + v * opi] = acc[nb][v]; else out[off + v * opi] = acc[nb][v] * sc;
            }
        }
    }
}

template <int NB, int MODE, bool T9>
__global__ __launch_bounds__(512, 1) void conv_dx_split_kernel(ConvDxArgs a)
{
    if (a.gate.closed()) return;
    conv_dx_split_body<NB, MODE, false, T9>(a, (int)blockIdx.x);
}

// The classes of a strided problem in one launch (ConvDxMulti).
template <int NB, int MODE>
__global__ __launch_bounds__(512, 1) void conv_dx_split_multi_kernel(ConvDxMulti m)
{
    if (m.cls[0].gate.closed()) return;
    int ci = 0;
    for (int i = 1; i < m.n; ++i) if ((int)blockIdx.x >= m.first[i]) ci = i;
    const ConvDxArgs a = m.cls[ci];
    conv_dx_split_body<NB, MODE, true, false>(a, (int)blockIdx.x - m.first[ci]);
}

// conv_dx_split.hip: mode MODE_BF16, MODE_BF16X2 or MODE_I8; nb 2, 4 or 7 pixel blocks a tile
hipError_t launch_conv_dx_split(int mode, const ConvDxArgs &args, int nb, int grid, int waves, size_t lds, hipStream_t s);
hipError_t launch_conv_dx_split(int mode, const ConvDxMulti &args, int nb, int grid, int waves, size_t lds, hipStream_t s);

}  // namespace dbp
