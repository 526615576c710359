// Host-side launchers of the matrix-core products: fully connected and implicit-im2col convolution,
// dithered (bf16x3 / int8) and dense (fp32) variants, with deterministic split-K.
#include <vector>
#include "conv_loaders.h"
#include "fc_kernel.h"
#include "fc2_kernel.h"
#include "fc_direct_kernel.h"
#include "fc2_i8_kernel.h"
#include "conv_dx_kernel.h"
#include "conv_dx_split_kernel.h"
#include "conv_dw_kernel.h"
#include "conv_dw_i8_kernel.h"
#include "conv_dwt_kernel.h"

namespace dbp {

namespace {

constexpr int kTargetWorkgroups = 512;          // two resident workgroups on each of the 256 CUs

struct Split { int n; int k_per; };

// Split the reduction so that tiles*n reaches kTargetWorkgroups, each part at least 4 K steps long
// and a multiple of `granule` (the K step, or one padded image for conv dW).
Split choose_split(int64_t tiles, int64_t K, int granule)
{
    int64_t want = (kTargetWorkgroups + tiles - 1) / tiles;
    int64_t units = (K + granule - 1) / granule;
    int64_t max_n = units / 4 > 0 ? units / 4 : 1;
    if (want > max_n) want = max_n;
    if (want < 1) want = 1;
    int64_t per = (units + want - 1) / want * granule;
    int64_t n = (K + per - 1) / per;
    return Split{(int)n, (int)per};
}

template <int MODE> constexpr int k_step() { return NCHUNK * ModeTraits<MODE>::KCH; }

template <int MODE, class AL, class BL, class OM>
hipError_t run_gemm(const AL &al, const BL &bl, const OM &om, int M, int N, int K, int granule, Scale scale,
                    typename ModeTraits<MODE>::Acc *out, void *scratch, size_t scratch_bytes, hipStream_t s)
{
    using Acc = typename ModeTraits<MODE>::Acc;
    GemmShape sh;
    sh.M = M; sh.N = N; sh.K = K;
    sh.tiles_m = (M + TM - 1) / TM;
    sh.tiles_n = (N + TN - 1) / TN;
    const int64_t tiles = (int64_t)sh.tiles_m * sh.tiles_n;
    Split sp = choose_split(tiles, K, granule);
    while (sp.n > 1 && (size_t)sp.n * M * N * sizeof(Acc) > scratch_bytes) {      // never exceed the workspace
        int64_t units = (K + granule - 1) / granule;
        int64_t n = sp.n - 1;
        sp.k_per = (int)((units + n - 1) / n * granule);
        sp.n = (int)((K + sp.k_per - 1) / sp.k_per);
    }
    sh.k_per_split = sp.n == 1 ? (K + granule - 1) / granule * granule : sp.k_per;
    dim3 grid((unsigned)tiles, 1, (unsigned)sp.n);
    hipLaunchKernelGGL((gemm_kernel<MODE, AL, BL, OM>), grid, dim3(256), 0, s, al, bl, om, sh, scale, out, (Acc *)scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (sp.n > 1) {
        int64_t total = (int64_t)M * N;
        int blocks = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
        hipLaunchKernelGGL((reduce_kernel<Acc, OM>), dim3(blocks), dim3(256), 0, s, (const Acc *)scratch, out, om, M, N, sp.n, scale);
        e = hipGetLastError();
    }
    return e;
}

// Weights re-laid for the dX product of a convolution: Wt[(r*S+s)*Kp + k][c] = W[k][c][r][s], zero for k >= K.
template <class T>
__global__ __launch_bounds__(256) void conv_weight_relayout_kernel(const T *W, T *Wt, ConvGeom g)
{
    const int64_t total = (int64_t)g.R * g.S * g.Kp * g.C;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int c = (int)(i % g.C);
        const int64_t kk = i / g.C;
        const int k = (int)(kk % g.Kp), rs = (int)(kk / g.Kp);
        Wt[i] = k < g.K ? W[((int64_t)k * g.C + c) * g.R * g.S + rs] : (T)0;
    }
}

ConvGeom make_geom(const ConvArgs &a, int kch, int kstep)
{
    ConvGeom g;
    g.N = (int)a.N; g.C = (int)a.C; g.H = (int)a.H; g.Wd = (int)a.Wd; g.K = (int)a.K; g.R = (int)a.R; g.S = (int)a.S;
    g.pad = (int)a.pad; g.st = (int)a.stride;
    g.P = (g.H + 2 * g.pad - g.R) / g.st + 1;
    g.Q = (g.Wd + 2 * g.pad - g.S) / g.st + 1;
    g.Kp = (g.K + kch - 1) / kch * kch;
    g.PQp = (g.P * g.Q + kstep - 1) / kstep * kstep;
    g.Ct = (int)a.ct(); g.Kt = (int)a.kt();
    return g;
}

size_t relayout_bytes(int64_t K, int64_t C, int64_t R, int64_t S)
{
    int64_t Kp = (K + 7) / 8 * 8;                       // multiple of every chunk length in use (4, 8)
    const size_t generic = (size_t)(R * S * Kp * C) * sizeof(float);
    // fast dX kernel: three bf16 planes, channels rounded to 32 on both sides
    const size_t fast = (size_t)(R * S) * ((K + 31) / 32 * 32) * ((C + 31) / 32 * 32) * 6;
    return align_up(generic > fast ? generic : fast, 256);
}

// Geometry of the fast dX kernel for one stride-1 problem (a whole layer, or one class of a strided layer), or
// ok == false when the generic kernel has to serve.  `k` arrives with the problem (N, C, H, Wd, K, R, S, pad, pad_w, P, Q
// and the output mapping) filled in; force_nb != 0 asks for that pixel-block count only.
struct ConvDxPlan { bool ok; int nb; ConvDxArgs args; size_t lds_bytes; int grid; int waves; float us; };   // waves: 0 conv_dx_kernel, else of conv_dx_split_kernel; us: modelled, of a workgroup

// Which of the two dX kernels, and with which tiles: by modelled time.  A workgroup costs its pairs (conv_dx_kernel: chunks) of k-groups,
// each its taps' matrix instructions and the staging of `items` fill items a lane, and its end; workgroups go over the chip's places
// in a row (two a CU, of eight wavefronts one), half a workgroup longer where they do not fit at once.  The constants (us) are fits over layers of 4 to
// 260 wide planes, 16 to 1024 channels, 1x1 to 7x7 taps and strides 1 to 3, with every form timed.  Time of the chosen form over the best form's,
// conv_dx_kernel alone over it, and how many layers were slower than on conv_dx_kernel (by 1.5 % or more):
//   fp32 weights            302 layers  1.016  1.59   3 (16 % at most)
//   two bf16 planes         306 layers  1.016  1.64   1 (15 %): chosen by the times of three planes; with the planes in the model as well 1.015, 1
//   int8 weights, stride 1  566 layers  1.020  1.81  11 (20 %)
//   int8 weights, strided   566 layers  1.019  1.41  14 (constants of stride 1, seven blocks allowed: 1.037, 63 layers, 38 %)
// (Fits and table are of conv_dx_kernel with 32x32x16 matrix instructions; with 16x16x32 it is up to a fifth faster, so that a layer near the line may be the
// other kernel's although conv_dx_kernel would now be the faster one; none is slower for it than it was.)
// Where the other kernel's time is `margin` times modelled, conv_dx_kernel keeps the layer; a wavefront without a pair would be idle.
struct ConvDxTimes { float block, tap, mma, staging, trip, base, spread, margin; };
static const ConvDxTimes &conv_dx_times(bool split, bool i8, bool strided)
{
    static const ConvDxTimes t[3][2] = {{{1.21f, 0.0f, 0.0725f, 0.05f, 0.28f, 7.5f, 1.19f, 1.0f}, {0.93f, 0.0635f, 0.0255f, 0.051f, 0.0f, 9.1f, 1.2f, 1.12f}},
                                        {{0.84f, 0.0f, 0.116f, 0.094f, 0.69f, 11.1f, 1.6f, 1.0f}, {0.76f, 0.095f, 0.0424f, 0.083f, 1.17f, 10.4f, 0.93f, 1.12f}},
                                        {{3.41f, 0.0f, 0.17f, 0.0709f, 0.0f, 0.0f, 0.78f, 1.0f}, {0.667f, 0.191f, 0.00534f, 0.0379f, 0.24f, 5.94f, 1.64f, 1.0f}}};
    return t[i8 ? (strided ? 2 : 1) : 0][split];
}

static float conv_dx_workgroup_us(const ConvDxArgs &k, int nb, int waves, int items, bool i8)
{
    const ConvDxTimes &t = conv_dx_times(waves != 0, i8, k.ost > 1);
    const float taps = (float)(k.R * k.S), mma = (float)(i8 ? nb : 3 * nb), staging = (float)(items * (i8 ? 16 : 8));
    const float trips = (float)(waves ? (k.pairs + waves - 1) / waves : k.n_chunks);
    return t.block * nb + trips * (taps * (t.tap + t.mma * mma) + t.staging * staging + t.trip);
}

// `longest`: of one workgroup; `sum`: of all of them.
static float conv_dx_launch_us(float longest, float sum, int64_t grid, int waves, size_t lds, bool i8, bool strided)
{
    const ConvDxTimes &t = conv_dx_times(waves != 0, i8, strided);
    const float slots = waves == 8 || lds > CDS_MAX_LDS / 2 ? 256.0f : 512.0f;
    const float all = sum / slots * t.spread + ((float)grid > slots ? 0.5f * longest : 0.0f);
    return (t.base + (longest > all ? longest : all)) * t.margin;
}

// The most patch rows, and dwords of one code plane, that a tile of `tile_px` consecutive pixels reads; false as soon as either is beyond what
// the caller has room for (large planes are refused at their first tile: a plan is made on the host in every call).  No division per tile:
// tile t begins in row h, column c (dbp_plan_auto_conv2d of a 3x3 layer, us, with divisions and to the end for every form / this: 112x112 8.6 / 5.8,
// 512x512 88 / 5.0, 2048x2048 1217 / 4.8).
static bool conv_dx_patch_extent(const ConvDxArgs &k, int tile_px, int tiles, int max_rows, int max_dw, int &prow, int &n_dw)
{
    const int rows = tile_px / k.Wd, cols = tile_px - rows * k.Wd;
    int h = 0, c = 0;
    prow = n_dw = 0;
    for (int t = 0; t < tiles; ++t) {
        const int end = c + cols - 1;                                // column of the tile's last pixel, counted from row h + rows
        const int h_last = t == tiles - 1 ? k.H - 1 : h + rows + (end >= k.Wd ? 1 : end < 0 ? -1 : 0);
        const int p_lo = h + k.pad - (k.R - 1);
        const int p_a = p_lo > 0 ? p_lo : 0, p_b = h_last + k.pad < k.P - 1 ? h_last + k.pad : k.P - 1;
        if (h_last - h + k.R > prow) prow = h_last - h + k.R;
        if (p_b >= p_a) {
            const int f_a = (p_a * k.Q) & ~3, d = ((p_b + 1) * k.Q - f_a + 3) >> 2;
            if (d > n_dw) n_dw = d;
        }
        if (prow > max_rows || n_dw > max_dw) return false;
        h += rows; c += cols;
        if (c >= k.Wd) { c -= k.Wd; ++h; }
    }
    return true;
}

static void conv_dx_plan_core(ConvDxPlan &pl, bool i8, int force_nb)
{
    ConvDxArgs &k = pl.args;
    pl.ok = false;
    k.PI = k.H * k.Wd; k.PQ = (k.P * k.Q + 3) / 4 * 4;           // the patch fill reads aligned dwords of a code plane: see conv_dx_codes
    if ((int64_t)(k.C + 32) * k.oPI >= ((int64_t)1 << 31)) return;   // 32-bit offsets inside one image
    k.Cp = (k.C + 31) / 32 * 32;
    const int chunk_k = CDX_KGC * (i8 ? 16 : 8);                 // reduction channels per chunk
    k.KG = (k.K + chunk_k - 1) / chunk_k * CDX_KGC;
    k.n_chunks = k.KG / CDX_KGC;
    const int ncb = k.Cp / 32;
    k.wc = ncb >= 3 ? 4 : ncb;
    k.wpx = 4 / k.wc;
    k.cgroups = (ncb + k.wc - 1) / k.wc;
    k.pw = k.Wd + k.S - 1;
    double best = -1.0;
    const int cand[3] = {7, 4, 2};
    for (int ci = 0; ci < 3; ++ci) {
        const int nb = cand[ci], tile_px = k.wpx * 32 * nb;
        if (force_nb && nb != force_nb) continue;
        const int tiles = (k.PI + tile_px - 1) / tile_px;
        int prow, n_dw;
        // both patch buffers in LDS, four k-groups each (and so their cell indices in 16 bits, 0xFFFF meaning "no cell"); the items of a lane
        static_assert(CDX_MAX_LDS / (2 * 16) < 0xFFFF, "cell indices");
        if (!conv_dx_patch_extent(k, tile_px, tiles, CDX_MAX_LDS / (2 * CDX_KGC * 16) / k.pw, 256 * CDX_ITMAX / CDX_KGC, prow, n_dw)) continue;
        const int64_t cells = (int64_t)prow * k.pw;
        const size_t lds = (size_t)2 * CDX_KGC * cells * 16;
        // time ~ rounds of workgroups over the chip (two resident per CU) x work per workgroup
        const int64_t grid = (int64_t)k.N * tiles * k.cgroups;
        const double cost = (double)nb * (double)((grid + 511) / 512);
        if (best < 0.0 || cost < best) {
            best = cost; pl.ok = true; pl.nb = nb; pl.waves = 0; pl.lds_bytes = lds; pl.us = conv_dx_workgroup_us(k, nb, 0, (n_dw * CDX_KGC + 255) / 256, i8);
            k.tiles = tiles; k.prow = prow; k.patch_cells = (int)cells;
        }
    }
    if (!pl.ok) return;
    const int64_t grid = (int64_t)k.N * k.tiles * k.cgroups;
    if (grid > 0x7FFFFFFF) { pl.ok = false; return; }
    pl.grid = (int)grid;
}

// Geometry of conv_dx_split_kernel for one stride-1 problem, likewise: 32*nb pixels and `waves` wavefronts a workgroup.
static void conv_dx_split_plan_core(ConvDxPlan &pl, bool i8, int nb, int waves)
{
    ConvDxArgs &k = pl.args;
    pl.ok = false;
    k.PI = k.H * k.Wd; k.PQ = (k.P * k.Q + 3) / 4 * 4;
    const int64_t img_out = k.dx_img + (int64_t)32 * k.oPI, img_codes = k.code_img;
    if (img_out >= ((int64_t)1 << 31) || img_codes >= ((int64_t)1 << 31)) return;
    const int G = i8 ? 16 : 8;
    k.Cp = (k.C + 31) / 32 * 32;
    k.KG = (k.K + CDX_KGC * G - 1) / (CDX_KGC * G) * CDX_KGC;
    k.n_chunks = k.KG / CDX_KGC;
    k.pairs = (k.K + 2 * G - 1) / (2 * G);
    k.wc = k.wpx = 1;
    k.cgroups = k.Cp / 32;
    k.pw = k.Wd + k.S - 1;
    const int tile_px = 32 * nb;
    k.NI = tile_px / k.PI;
    if (k.NI > k.N) k.NI = k.N;
    if (k.NI < 1) k.NI = 1;
    k.tiles = k.NI > 1 ? 1 : (k.PI + tile_px - 1) / tile_px;
    if (k.pairs < waves) return;                                     // a wavefront would have nothing to do
    int prow, n_dw;
    if (!conv_dx_patch_extent(k, tile_px, k.tiles, CDS_MAX_LDS / (2 * 16 * waves) / k.pw, 64 * cds_items(nb) / 2, prow, n_dw)) return;
    if (k.NI > 1 && 2 * k.NI * n_dw > 64 * cds_items(nb)) k.NI = 64 * cds_items(nb) / (2 * n_dw);
    while (k.NI > 1 && (k.NI * img_codes >= ((int64_t)1 << 31) || k.NI * img_out >= ((int64_t)1 << 31))) --k.NI;
    k.prow = prow; k.img_cells = prow * k.pw; k.patch_cells = k.NI * k.img_cells; k.wave_cells = 2 * k.patch_cells + 1;
    const int64_t stage = (int64_t)waves * k.wave_cells * 16, fold = (int64_t)waves * nb * 8 * 64 * 4, lds = stage > fold ? stage : fold;
    if (lds > CDS_MAX_LDS || k.wave_cells >= 0xFFFF) return;
    const int64_t grid = (int64_t)((k.N + k.NI - 1) / k.NI) * k.tiles * k.cgroups;
    if (grid > 0x7FFFFFFF) return;
    pl.ok = true; pl.nb = nb; pl.waves = waves; pl.lds_bytes = (size_t)lds; pl.grid = (int)grid;
    pl.us = conv_dx_workgroup_us(k, nb, waves, (2 * k.NI * n_dw + 63) / 64, i8);
}

// The pixel blocks and wavefronts that conv_dx_split_kernel runs with.
static const struct { int nb, waves; } kDxSplitForms[6] = {{7, 4}, {4, 4}, {2, 4}, {7, 8}, {4, 8}, {2, 8}};

ConvDxPlan conv_dx_plan(const ConvArgs &a, bool i8 = false)
{
    ConvDxPlan pl{};
    ConvDxArgs &k = pl.args;
    if (a.stride != 1) return pl;                                // strided layers: conv_dx_strided_plan
    k.N = (int)a.N; k.C = (int)a.C; k.H = (int)a.H; k.Wd = (int)a.Wd; k.K = (int)a.K; k.R = (int)a.R; k.S = (int)a.S;
    k.pad = (int)a.pad; k.pad_w = (int)a.pad;
    k.code_img = a.kt() * ((a.H + 2 * a.pad - a.R + 1) * (a.Wd + 2 * a.pad - a.S + 1) + 3); k.dx_img = a.ct() * a.H * a.Wd;   // upper bounds until the launch
    k.P = k.H + 2 * k.pad - k.R + 1; k.Q = k.Wd + 2 * k.pad - k.S + 1;
    k.oW = k.Wd; k.oPI = k.H * k.Wd; k.ost = 1; k.oh0 = 0; k.ow0 = 0;
    conv_dx_plan_core(pl, i8, 0);
    float best = pl.ok ? conv_dx_launch_us(pl.us, pl.us * (float)pl.grid, pl.grid, 0, pl.lds_bytes, i8, false) : 3.0e38f;
    for (const auto &f : kDxSplitForms) {
        ConvDxPlan sp = pl;
        conv_dx_split_plan_core(sp, i8, f.nb, f.waves);
        const float us = sp.ok ? conv_dx_launch_us(sp.us, sp.us * (float)sp.grid, sp.grid, f.waves, sp.lds_bytes, i8, false) : 3.0e38f;
        if (sp.ok && us < best) { best = us; pl = sp; }
    }
    return pl;
}

// A strided layer as st*st stride-1 problems, one per class of output pixels (h mod st, w mod st): class (ph, pw) has
// the taps r = r0 + st*t, r0 = (ph + pad) mod st, and reads code row i + (ph + pad - r0)/st - t for its output row i.
// Classes without taps (a 1x1 kernel with stride 2 has three) are all zero: `zero_fill` asks for dX to be cleared first.
struct ConvDxStridedPlan { bool ok, zero_fill; int nb; ConvDxMulti multi; CdxTapMap map; int taps, tap_base[CDX_MAX_CLASSES]; size_t lds_bytes; int grid, waves; };

ConvDxStridedPlan conv_dx_strided_plan(const ConvArgs &a, bool i8)
{
    ConvDxStridedPlan sp{};
    const int st = (int)a.stride, R = (int)a.R, S = (int)a.S, pad = (int)a.pad, H = (int)a.H, Wd = (int)a.Wd;
    if (st < 2 || st * st > CDX_MAX_CLASSES || R * S > 64) return sp;
    const int P = (H + 2 * pad - R) / st + 1, Q = (Wd + 2 * pad - S) / st + 1;
    // One pixel-block count for all classes (one launch): conv_dx_kernel's with the least rounds x work per workgroup, and then the faster
    // kernel (conv_dx_workgroup_us).
    ConvDxStridedPlan best{};
    double best_cost = -1.0;
    float best_us = 3.0e38f;
    const int cand[3] = {7, 4, 2};
    for (int attempt = 0; attempt < 9; ++attempt) {
        const bool split = attempt >= 3;
        const int nb = split ? kDxSplitForms[attempt - 3].nb : cand[attempt];
        sp.waves = split ? kDxSplitForms[attempt - 3].waves : 0;
        if (split && i8 && nb == 7) continue;                    // (conv_dx_split.hip)
        float longest = 0.0f, sum = 0.0f;
        sp.ok = false;
        bool all = true;
        sp.multi.n = 0; sp.taps = 0; sp.zero_fill = false; sp.lds_bytes = 0;
        int64_t grid = 0;
        for (int ph = 0; ph < st && all; ++ph) {
            for (int pw = 0; pw < st && all; ++pw) {
                const int Hv = ph < H ? (H - ph + st - 1) / st : 0, Wv = pw < Wd ? (Wd - pw + st - 1) / st : 0;
                if (Hv == 0 || Wv == 0) continue;                // no such pixels
                const int r0 = (ph + pad) % st, s0 = (pw + pad) % st;
                const int Rv = r0 < R ? (R - r0 + st - 1) / st : 0, Sv = s0 < S ? (S - s0 + st - 1) / st : 0;
                if (Rv == 0 || Sv == 0) { sp.zero_fill = true; continue; }
                ConvDxPlan pl{};
                ConvDxArgs &k = pl.args;
                k.N = (int)a.N; k.C = (int)a.C; k.H = Hv; k.Wd = Wv; k.K = (int)a.K; k.R = Rv; k.S = Sv;
                k.pad = (ph + pad - r0) / st; k.pad_w = (pw + pad - s0) / st;
                k.P = P; k.Q = Q;
                k.code_img = a.kt() * ((int64_t)P * Q + 3); k.dx_img = a.ct() * H * Wd;          // upper bounds until the launch
                k.oW = Wd; k.oPI = H * Wd; k.ost = st; k.oh0 = ph; k.ow0 = pw;
                if (split) conv_dx_split_plan_core(pl, i8, nb, sp.waves); else conv_dx_plan_core(pl, i8, nb);
                if (!pl.ok) { all = false; break; }
                // this class's prepared taps follow the earlier classes'
                for (int t = 0; t < Rv; ++t)
                    for (int u = 0; u < Sv; ++u) sp.map.real[sp.taps + t * Sv + u] = (uint8_t)((r0 + st * t) * S + (s0 + st * u));
                k.codes = nullptr; k.wp = nullptr; k.dX = nullptr; k.scale = Scale{1.0f, nullptr};   // set at the launch
                sp.multi.cls[sp.multi.n] = k;
                sp.multi.first[sp.multi.n] = (int)grid;
                sp.tap_base[sp.multi.n] = sp.taps;
                sp.taps += Rv * Sv;
                grid += pl.grid;
                sum += pl.us * (float)pl.grid;
                if (pl.us > longest) longest = pl.us;
                if (pl.lds_bytes > sp.lds_bytes) sp.lds_bytes = pl.lds_bytes;
                ++sp.multi.n;
            }
        }
        if (!all || grid > 0x7FFFFFFF) continue;
        sp.multi.first[sp.multi.n] = (int)grid;
        sp.ok = true; sp.nb = nb; sp.grid = (int)grid;
        const double cost = (double)nb * (double)((grid + 511) / 512);
        const float us = conv_dx_launch_us(longest, sum, grid, sp.waves, sp.lds_bytes, i8, true);
        if (split ? us < best_us : best_cost < 0.0 || cost < best_cost) { best_cost = cost; best_us = us; best = sp; }
    }
    if (best_us > 2.0e38f) { sp.ok = false; return sp; }
    sp = best;
    for (int t = sp.taps; t < 64; ++t) sp.map.real[t] = 0;
    return sp;
}


// Geometry of the fast dW kernel (conv_dw_kernel.h), or ok == false when the generic kernel has to serve.
struct ConvDwPlan { bool ok; int mb; ConvDwArgs args; size_t lds_bytes, partial_bytes; int grid, reduce_grid; };

ConvDwPlan conv_dw_plan(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t pad, bool i8)
{
    ConvDwPlan pl;
    pl.ok = false; pl.partial_bytes = 0; pl.lds_bytes = 0;
    ConvDwArgs &k = pl.args;
    // one accumulator per tap: compiled tap counts only.  (A 1x1 instantiation was measured: a single tap
    // leaves the stagers far behind the matrix cores, and the generic kernel is faster there.)
    if (!(R == 3 && S == 3)) return pl;
    if (pad > 1) return pl;                                          // compiled paddings: 0 and 1
    const int64_t P = H + 2 * pad - R + 1, Q = Wd + 2 * pad - S + 1;
    if ((H * Wd) % 4 || (P * Q) % 4) return pl;                     // rows are fetched as aligned 4-element pieces
    if (C * H * Wd >= ((int64_t)1 << 29) || K * P * Q >= ((int64_t)1 << 29) || K * C * R * S >= ((int64_t)1 << 31)) return pl;
    k.N = (int)N; k.C = (int)C; k.H = (int)H; k.Wd = (int)Wd; k.K = (int)K; k.P = (int)P; k.Q = (int)Q; k.pad = (int)pad;
    k.Ct = k.C; k.Kt = k.K;                                          // one group of a grouped layer: set at the launch
    const int FRAG = i8 ? 16 : 8, KSTEP = 2 * FRAG, ESZ = i8 ? 1 : 2, PL = i8 ? 1 : 3, CQL = 128, XQL = 64;
    int64_t pw = Wd + pad;
    const int64_t over = S - 1 - pad > 0 ? S - 1 - pad : 0;
    if (Q + over > pw) pw = Q + over;
    pw = (pw + FRAG - 1) / FRAG * FRAG;
    if (pw > 256) return pl;
    k.PW = (int)pw;
    const int t_max = CDW_M8 + (int)((R - 1) * pw + pad);
    double best = -1.0;
    for (int mb = 1; mb >= 1 && !pl.ok; --mb) {
        const int TK = 64 * mb, TC = 64;
        for (int ru = 1; ru <= H && ru * Wd <= 4 * XQL - 9 && ru * pw <= 320; ++ru) {
            const int tpc = (int)(ru * pw);
            if (tpc % KSTEP) continue;
            const int len = (tpc + t_max + FRAG + 3) / 4 * 4;
            const int nr = (int)((len - CDW_M8 - 1) / pw) + 2;
            const int nqc = (int)((nr * Q + 9) / 4), nqx = (int)((ru * Wd + 9) / 4);
            if (nqc > CQL || nqx > XQL) continue;
            int xc = tpc / FRAG; if (xc % 2 == 0) ++xc;              // odd cell counts spread a fragment read over the banks
            int cc = (len + FRAG - 1) / FRAG; if (cc % 2 == 0) ++cc;
            const size_t lds = 2 * ((size_t)PL * TC * xc * FRAG * ESZ + (size_t)TK * cc * FRAG * ESZ);   // double buffered
            if (lds > (size_t)CDW_MAX_LDS) continue;
            const int chunks = (int)((H + ru - 1) / ru);
            const double cost = (double)chunks * (tpc + 64.0);      // matrix-core steps plus a fixed cost per unit
            if (best < 0.0 || cost < best) {
                best = cost; pl.ok = true; pl.mb = mb; pl.lds_bytes = lds;
                k.RU = ru; k.TPc = tpc; k.chunks = chunks; k.lenC = len; k.pitchX = xc * FRAG; k.pitchC = cc * FRAG;
                k.NR = nr; k.nqx = nqx; k.nqc = nqc; k.lds_cells = (int)(lds / 16);
            }
        }
    }
    if (!pl.ok) return pl;
    k.row4x = Wd % 4 == 0; k.row4c = Q % 4 == 0;
    k.row2x = Wd % 2 == 0; k.row2c = Q % 2 == 0;
    // code rows of whole 8-code pieces under the whole-piece staging path (bf16 modes): half as many, twice as wide code loads
    k.c8 = !i8 && k.row4x && k.row4c && Q % 8 == 0;
    if (k.c8) k.nqc = (k.nqc + 1) / 2;
    k.xshift = k.nqx <= 16 ? 4 : k.nqx <= 32 ? 5 : 6;
    k.cshift = k.nqc <= 32 ? 5 : k.nqc <= 64 ? 6 : 7;
    const int TK = 64 * pl.mb;
    k.tiles_k = (int)((K + TK - 1) / TK); k.tiles_c = (int)((C + 63) / 64);
    const int64_t tiles = (int64_t)k.tiles_k * k.tiles_c;
    const int64_t units = N * k.chunks;
    if (units >= ((int64_t)1 << 31) || tiles > 65535) { pl.ok = false; return pl; }
    k.units = (int)units;
    int64_t want = tiles >= 256 ? 1 : 256 / tiles;                   // one workgroup per CU
    if (want > units) want = units;
    k.units_per_split = (int)((units + want - 1) / want);
    k.n_split = (int)((units + k.units_per_split - 1) / k.units_per_split);
    const int64_t ne = R * S * pl.mb * 16;
    pl.partial_bytes = k.n_split > 1 ? (size_t)tiles * k.n_split * ne * 256 * 4 : 0;
    pl.grid = (int)(tiles * k.n_split);
    pl.reduce_grid = (int)(tiles * (ne / 4) * 16);                  // (tile, group of 4 elements, 16 of the 256 slots)
    return pl;
}

// Geometry of the int8 3x3 dW kernel with transposed cells (conv_dw_i8_kernel.h); ok == false when it does not apply.
struct ConvDwI8Plan { bool ok; ConvDwI8Args args; size_t lds_bytes, partial_bytes; int grid, reduce_grid; };

ConvDwI8Plan conv_dw_i8_plan(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t pad)
{
    ConvDwI8Plan pl;
    pl.ok = false; pl.partial_bytes = 0; pl.lds_bytes = 0;
    ConvDwI8Args &k = pl.args;
    if (!(R == 3 && S == 3 && pad == 1)) return pl;
    if (Wd % 4 || Wd < 16 || Wd > 224 || H < 1) return pl;           // 16-byte loads at dword-aligned addresses inside a row
    if (H * Wd >= ((int64_t)1 << 24) || K * C * 9 >= ((int64_t)1 << 31)) return pl;   // 64 channels of a tile: 32-bit offsets
    const int pw = (int)((Wd + 1 + 15) / 16 * 16), cpr = pw / 16, dc = (int)((Wd + 15) / 16);
    double best = -1.0;
    for (int ru = 1; ru <= H; ++ru) {
        const int xpairs = ru * dc, cpairs = (ru + 2) * dc;
        if (cpairs > 64) break;                                      // 256 stager threads cover >= 4 channels a pass, 16 passes at most
        const int n_steps = (ru * cpr + 1) / 2;
        const int xcells = (2 * n_steps) | 1;                        // odd: a fragment read spreads over the banks
        int ccells = (ru + 2) * cpr + 2;                             // the patch and a zero cell at either end
        if (ccells < 2 * n_steps + 2 * cpr + 2) ccells = 2 * n_steps + 2 * cpr + 2;   // the last step's reach
        ccells |= 1;
        const size_t lds = 2 * (size_t)64 * (xcells + ccells) * 16 + 256 * 16;   // two buffers and a spare cell per stager thread
        if (lds > (size_t)CDW_MAX_LDS) break;
        const int chunks = (int)((H + ru - 1) / ru);
        const double cost = (double)chunks * (n_steps + 1.5);       // matrix-core steps plus a fixed cost per unit
        if (best < 0.0 || cost < best) {
            best = cost; pl.ok = true; pl.lds_bytes = lds;
            k.RU = ru; k.chunks = chunks; k.n_steps = n_steps; k.xcells = xcells; k.ccells = ccells;
            k.xpairs = xpairs; k.cpairs = cpairs; k.lds_cells = (int)(lds / 16) - 256;
        }
    }
    if (!pl.ok) return pl;
    k.N = (int)N; k.C = (int)C; k.H = (int)H; k.Wd = (int)Wd; k.K = (int)K; k.PW = pw; k.CPR = cpr; k.DC = dc;
    k.Ct = k.C; k.Kt = k.K;
    k.tiles_k = (int)((K + 63) / 64); k.tiles_c = (int)((C + 63) / 64);
    const int64_t tiles = (int64_t)k.tiles_k * k.tiles_c, units = N * k.chunks;
    if (units >= ((int64_t)1 << 31) || tiles > 65535) { pl.ok = false; return pl; }
    k.units = (int)units;
    int64_t want = tiles >= 256 ? 1 : 256 / tiles;                   // one workgroup per CU
    if (want > units) want = units;
    k.units_per_split = (int)((units + want - 1) / want);
    k.n_split = (int)((units + k.units_per_split - 1) / k.units_per_split);
    pl.partial_bytes = k.n_split > 1 ? (size_t)tiles * k.n_split * 144 * 256 * 4 : 0;
    pl.grid = (int)(tiles * k.n_split);
    pl.reduce_grid = (int)(tiles * 36 * 16);                         // (tile, group of 4 accumulator elements, 16 of the 256 slots)
    return pl;
}

hipError_t launch_conv_dw_i8(const ConvDwI8Plan &pl, hipStream_t s)
{
    static bool raised = false;                                      // more than 64 KiB of dynamic LDS: allowed per kernel, once
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_dw_i8_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, CDW_MAX_LDS);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL(conv_dw_i8_kernel, dim3(pl.grid), dim3(512), pl.lds_bytes, s, pl.args);
    if (pl.args.n_split > 1) {
        ConvDwArgs r{};                                              // the reduction reads the partial layout of both dW kernels
        r.partial = pl.args.partial; r.dW = pl.args.dW; r.n_split = pl.args.n_split; r.tiles_k = pl.args.tiles_k;
        r.K = pl.args.K; r.C = pl.args.C; r.scale = Scale{1.0f, nullptr}; r.gate = pl.args.gate;
        hipLaunchKernelGGL((conv_dw_reduce_kernel<MODE_I8, 3, 3, 1>), dim3(pl.reduce_grid), dim3(256), 0, s, r);
    }
    return hipGetLastError();
}

// Geometry of the general dW kernel (conv_dwt_kernel.h), or ok == false when it does not apply (more than 4096 taps, frames that do not
// fit, 32-bit offsets).
struct ConvDwtPlan { bool ok; int G, waves, grid, reduce_grid, tch, tap_chunks, zg; ConvDwtArgs args; size_t lds_bytes, partial_bytes, reduce_lds; float us; };

ConvDwtPlan conv_dwt_plan(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t pad, int64_t stride, bool i8, int planes)
{
    ConvDwtPlan pl;
    pl.ok = false; pl.partial_bytes = 0;
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1, T = R * S;
    const int RUN = DWT_RUN(i8), pitch = (i8 ? 32 : 64 * planes) + 8;
    if (T > 4096 || C * H * Wd >= ((int64_t)1 << 29) || K * P * Q >= ((int64_t)1 << 29) || K * C * T >= ((int64_t)1 << 30)) return pl;
    ConvDwtArgs &k = pl.args;
    k.N = (int)N; k.C = (int)C; k.H = (int)H; k.Wd = (int)Wd; k.K = (int)K; k.S = (int)S; k.T = (int)T; k.st = (int)stride; k.pad = (int)pad;
    k.P = (int)P; k.Q = (int)Q; k.Ct = k.C; k.Kt = k.K; k.tiny = P * Q < RUN ? 1 : 0;
    // One tap: a wavefront takes several blocks of input channels.  Else taps per wavefront: 3 (up to 12 wavefronts) or 4 (8), whichever
    // keeps more of the matrix instructions on real taps and the wavefronts even over the four SIMDs.
    double best = -1.0;
    int m = 8;
    const bool one = T == 1;
    const int st_lds = one ? 1 : (int)stride;
    k.st_load = one ? (int)stride : 1; k.st_lds = st_lds;
    if (one) { pl.G = C > 64 ? 4 : 2; k.tap_blocks = 1; k.tg = 1; }
    for (int G = 3; G <= 4 && !one; ++G) {
        const int most = G == 3 ? 12 : 8, groups = (int)((T + G - 1) / G), blocks = (groups + most - 1) / most, tg = (groups + blocks - 1) / blocks;
        int mm = 1;
        while (2 * mm * tg <= most) mm *= 2;
        const int waves = mm * tg;
        const double eff = (double)T / ((double)G * tg * blocks) * waves / ((waves + 3) / 4 * 4);
        if (eff > best) { best = eff; pl.G = G; k.tap_blocks = blocks; k.tg = tg; m = mm; }
    }
    const int MF = pl.G == 2 ? 4 : 2, gc = one ? pl.G : 1;                   // gc: blocks of input channels of a wavefront
    const int items = one ? 6 : 4, citems = (one ? 16 : pl.G == 3 ? 8 : 12) / (RUN / 4);
    pl.waves = m * k.tg;
    // The rest of the wavefronts along output channels (an activation is then staged for more of them), input channels, or steps
    // (fewer partial sums); units: whole images (several small ones), bands of rows, or bands of rows and columns.  By modelled
    // time: a step keeps the four SIMDs busy for its matrix instructions, a chunk of staged pixels (halos included) costs about
    // 600 cycles, a unit 1500 more; partial sums are written and read at about 4.5 TB/s.
    best = -1.0;
    int64_t best_units = 0;
    const double t_step = (double)pl.waves / 4.0 * MF * pl.G * 32.0 * (i8 ? 1 : planes);
    const int widths[8] = {(int)Q, 4, 8, 16, 32, 48, 64, 96};
    for (int kg = 1; kg <= m; kg *= 2)
        for (int cb = 1; kg * cb <= m; cb *= 2) {
            const int kt = 32 * MF * kg, ps = m / (kg * cb);
            const int blocks = cb * gc;
            if ((kg > 1 && kt / 2 >= K) || (cb > 1 && 16 * blocks >= C)) continue;         // half of the tile would be empty
            int max_chunks = items * pl.waves / (8 * blocks);
            const int fit = (int)((DWT_MAX_LDS - 4096) / ((size_t)64 * (2 * pitch * blocks)));
            if (max_chunks > fit) max_chunks = fit;
            const int max_px = 64 * max_chunks;
            const int64_t tk = (K + kt - 1) / kt, tc = (C + 32 * blocks - 1) / (32 * blocks), tiles = tk * tc * k.tap_blocks;
            for (int wi = 0; wi < 8; ++wi) {
                const int qb = widths[wi];
                if (wi > 0 && (qb >= Q || k.tiny)) break;
                const int fw = (int)((qb - 1) * st_lds + S);
                if ((int)R * fw > max_px) continue;
                const int cbands = (int)((Q + qb - 1) / qb);
                const bool flat = wi == 0;
                int pb = (int)((max_px / fw - R) / st_lds + 1), bands = 0, ni = 1, frame = 0, runs_row = 0, runs_img = 0, steps = 0, chunks = 0;
                size_t lds = 0;
                int tables = 1, last_rows = 0;
                const int last_cols = (int)Q - (cbands - 1) * qb;
                if (pb > P) pb = (int)P;
                bool fits = false;
                for (; pb >= 1 && !fits; --pb) {                             // the tallest band (then the most images) whose codes fit beside it
                    bands = (int)((P + pb - 1) / pb);
                    pb = (int)((P + bands - 1) / bands);
                    frame = (int)((pb - 1) * st_lds + R) * fw;
                    last_rows = (int)P - (bands - 1) * pb;
                    tables = i8 ? 1 : (last_rows < pb ? 2 : 1) * (last_cols < qb ? 2 : 1);     // (integers have no NaN)
                    ni = 1;
                    if (flat && bands == 1) {
                        ni = max_px / frame;
                        const int64_t keep = N * tiles / 256;             // no more images a unit than leave every CU a unit
                        if (ni > keep) ni = keep < 1 ? 1 : (int)keep;
                        if (ni > 127) ni = 127;
                    }
                    runs_row = flat ? (pb * qb + RUN - 1) / RUN : (qb + RUN - 1) / RUN; runs_img = flat ? runs_row : runs_row * pb;
                    for (; ni >= 1 && !fits; --ni) {
                        steps = (runs_img * ni + 1) / 2; chunks = (frame * ni + 63) / 64;
                        lds = 2 * ((size_t)chunks * 64 * pitch * blocks + (size_t)kt * (2 * steps + 1) * RUN) + (size_t)steps * RUN * 8 * tables;
                        fits = lds <= (size_t)DWT_MAX_LDS && chunks <= pl.waves && pl.waves / chunks * items >= 8 * blocks && 2 * steps <= 64 * pl.waves && kt <= citems * (64 * pl.waves / (2 * steps));
                        if (fits) break;
                    }
                    if (fits) break;
                }
                if (!fits) continue;
                const int64_t units = (N + ni - 1) / ni * bands * cbands;
                int64_t want = tiles >= 256 ? 1 : 256 / tiles;             // one workgroup per CU
                if (want > units) want = units;
                const int64_t per = (units + want - 1) / want, ns = (units + per - 1) / per;
                const double rounds = (double)((tiles * ns + 255) / 256);
                double us = rounds * (double)per * ((double)((steps + ps - 1) / ps) * t_step + chunks * blocks * 600.0 + 1500.0) / 2000.0;
                if (tables > 1) us *= 1.04;                                // (the pixel table chosen per unit)
                if (ns > 1) us += 4.0 + (double)tiles * ns * (pl.waves / ps) * MF * pl.G * 4096.0 * 2.0 / 4.5e6;
                if (best >= 0.0 && us >= best) continue;
                best = us; best_units = units;
                k.kg = kg; k.cb = cb; k.ps = ps; k.tiles_k = (int)tk; k.tiles_c = (int)tc;
                k.PB = pb; k.bands = bands; k.QB = qb; k.cbands = cbands; k.NI = ni; k.frame_w = fw; k.frame = frame; k.chunks = chunks;
                k.runs_row = runs_row; k.runs_img = runs_img; k.steps = steps; k.flat = flat ? 1 : 0;
                k.last_rows = last_rows; k.last_cols = last_cols; k.tables = tables;
                k.table_row = tables > 1 && last_rows < pb ? 2 * steps * RUN : 0; k.table_col = tables > 1 && last_cols < qb ? tables * steps * RUN : 0;
                k.blocks = blocks; k.x_bytes = chunks * 64 * pitch * blocks; k.buf_bytes = k.x_bytes + kt * (2 * steps + 1) * RUN;
                k.code_step = 64 * pl.waves / (2 * steps); pl.lds_bytes = lds;
                k.units_per_split = (int)per; k.n_split = (int)ns;
            }
        }
    if (best < 0.0) return pl;
    pl.us = (float)best;
    const int64_t tiles = (int64_t)k.tiles_k * k.tiles_c * k.tap_blocks;
    if (best_units >= ((int64_t)1 << 30) || tiles > 65535 || (int64_t)k.NI * k.K * P * Q >= ((int64_t)1 << 30) || (int64_t)k.NI * C * H * Wd >= ((int64_t)1 << 29)) return pl;
    k.units = (int)best_units;
    const size_t wave_bytes = (size_t)MF * pl.G * 4096;
    const int tile_waves = k.tg * k.cb * k.kg;
    pl.partial_bytes = k.n_split > 1 ? (size_t)tiles * k.n_split * tile_waves * wave_bytes : 0;
    const size_t fold = (size_t)(k.ps / 2) * tile_waves * wave_bytes;
    if (fold > pl.lds_bytes) pl.lds_bytes = fold;
    if (pl.lds_bytes > (size_t)DWT_MAX_LDS) return pl;
    pl.grid = (int)(tiles * k.n_split);
    // taps per workgroup of the reduction: all of them, fewer while the chip has room (never below 4 where there are as many)
    const int red = k.tiles_k * k.tiles_c * k.kg * k.blocks * MF * 4;
    pl.tch = (int)(T < 60 ? T : 60);                                        // (64 of them fill the default LDS of a workgroup)
    while (pl.tch > 4 && red * ((T + pl.tch - 1) / pl.tch) < 256) pl.tch = (pl.tch + 1) / 2;
    pl.tap_chunks = (int)((T + pl.tch - 1) / pl.tch);
    pl.reduce_grid = red * pl.tap_chunks;
    pl.zg = 16 / pl.tch < (k.n_split + 3) / 4 ? 16 / pl.tch : (k.n_split + 3) / 4;      // groups of threads: at least four splits each
    if (pl.zg < 1) pl.zg = 1;
    pl.reduce_lds = (size_t)pl.zg * 64 * pl.tch * 16;
    pl.ok = true;
    return pl;
}

// Modelled time of dW on the generic kernel for layers of few input channels: a K step takes 4.4 us (int8, twice as deep, 9.4) with its loads and their checks, rounds of two
// workgroups a CU, partial sums at 4.5 TB/s.  Within 17 % of 280 layers of up to 64 input channels.
float conv_dw_generic_us(int64_t N, int64_t C, int64_t P, int64_t Q, int64_t K, int64_t taps, bool i8)
{
    const int step = i8 ? k_step<MODE_I8>() : k_step<MODE_BF16>(), cell = i8 ? 16 : 8;
    const int64_t outputs = K * C * taps, tiles = ((K + TM - 1) / TM) * ((C * taps + TN - 1) / TN), Kred = N * ((P * Q + cell - 1) / cell * cell);
    const Split sp = choose_split(tiles, Kred, step);
    const float wgs = (float)tiles * sp.n / 256.0f, rounds = wgs > 2.0f ? wgs / 2.0f : 1.0f, steps = rounds * (float)(((sp.n > 1 ? sp.k_per : Kred) + step - 1) / step);
    return (i8 ? 4.6f + 9.4f * steps : 3.3f + 4.4f * steps) + (i8 ? 11.3f : 8.4f) * (wgs < 2.0f ? wgs : 2.0f) +
           (sp.n > 1 ? (i8 ? 4.2f : 2.0f) + (float)sp.n * outputs * 8.0f / 4.5e6f : 0.0f) + (i8 ? 0.0f : 2.9e-5f * outputs);
}

template <bool I8, int PL, int G, bool ONE, bool RAGGED>
hipError_t launch_conv_dwt_as(const ConvDwtPlan &pl, hipStream_t s)
{
    static bool raised = false;                                      // more than 64 KiB of dynamic LDS: allowed per kernel, once
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_dwt_kernel<I8, PL, G, ONE, RAGGED>), hipFuncAttributeMaxDynamicSharedMemorySize, DWT_MAX_LDS);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL((conv_dwt_kernel<I8, PL, G, ONE, RAGGED>), dim3(pl.grid), dim3(64 * pl.waves), pl.lds_bytes, s, pl.args);
    if (pl.args.n_split > 1)
        hipLaunchKernelGGL((conv_dwt_reduce_kernel<G, ONE>), dim3(pl.reduce_grid), dim3(64 * pl.tch * pl.zg < 1024 ? 64 * pl.tch * pl.zg : 1024), pl.reduce_lds, s, pl.args, I8 ? 1 : 0,
                           pl.tch, pl.tap_chunks, pl.zg);
    return hipGetLastError();
}

template <bool I8, int PL, bool RAGGED>
hipError_t launch_conv_dwt_of(const ConvDwtPlan &pl, hipStream_t s)
{
    if (pl.args.T == 1) return pl.G == 2 ? launch_conv_dwt_as<I8, PL, 2, true, RAGGED>(pl, s) : launch_conv_dwt_as<I8, PL, 4, true, RAGGED>(pl, s);
    return pl.G == 3 ? launch_conv_dwt_as<I8, PL, 3, false, RAGGED>(pl, s) : launch_conv_dwt_as<I8, PL, 4, false, RAGGED>(pl, s);
}

template <bool I8, int PL>
hipError_t launch_conv_dwt(const ConvDwtPlan &pl, hipStream_t s)
{
    if constexpr (!I8) { if (pl.args.tables > 1) return launch_conv_dwt_of<I8, PL, true>(pl, s); }
    return launch_conv_dwt_of<I8, PL, false>(pl, s);
}

template <int MODE, int R, int S, int PAD, int MB, int ROWS>
hipError_t launch_conv_dw_fast_as(const ConvDwPlan &pl, hipStream_t s)
{
    // more than 64 KiB of dynamic LDS has to be allowed per kernel, once
    static bool raised = false;
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_dw_kernel<MODE, R, S, PAD, MB, ROWS>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, CDW_MAX_LDS);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL((conv_dw_kernel<MODE, R, S, PAD, MB, ROWS>), dim3(pl.grid), dim3(512), pl.lds_bytes, s, pl.args);
    if (pl.args.n_split > 1)
        hipLaunchKernelGGL((conv_dw_reduce_kernel<MODE, R, S, MB>), dim3(pl.reduce_grid), dim3(256), 0, s, pl.args);
    return hipGetLastError();
}

template <int MODE, int R, int S, int PAD, int MB>
hipError_t launch_conv_dw_fast(const ConvDwPlan &pl, hipStream_t s)
{
    // rows that are whole numbers of aligned 4-element pieces have a staging path of their own
    // (and code rows of whole 8-code pieces, bf16 modes, one that loads the codes 8 bytes at a time)
    if constexpr (MODE != MODE_I8) {
        if (pl.args.c8) return launch_conv_dw_fast_as<MODE, R, S, PAD, MB, 2>(pl, s);
    }
    return pl.args.row4x && pl.args.row4c ? launch_conv_dw_fast_as<MODE, R, S, PAD, MB, 1>(pl, s)
                                          : launch_conv_dw_fast_as<MODE, R, S, PAD, MB, 0>(pl, s);
}

// ---- fully connected products with staging and multiplying wavefronts (fc2_kernel.h, fc2_i8_kernel.h) -----------
struct FcPlan { int tiles_m, tiles_n, n_split, k_per_split; int64_t tiles; size_t partial_bytes; };

// Plans of the two products for the kernel with staging and multiplying wavefronts: reductions are split
// into items of about half a workgroup's share of all K steps (one workgroup per CU), at least 8 steps.
void fc2_plans(int64_t B, int64_t in, int64_t out, bool want_dx, bool want_dw, FcPlan &dx, FcPlan &dw, int kt = FC2_KT)
{
    auto base = [kt](int64_t M, int64_t N, int64_t K, FcPlan &pl) {
        pl.tiles_m = (int)((M + FC2_TM - 1) / FC2_TM);
        pl.tiles_n = (int)((N + FC2_TN - 1) / FC2_TN);
        pl.tiles = (int64_t)pl.tiles_m * pl.tiles_n;
        return (K + kt - 1) / kt;
    };
    const int64_t sx = base(B, in, out, dx), sw = base(out, in, B, dw);
    const int64_t all = (want_dx ? dx.tiles * sx : 0) + (want_dw ? dw.tiles * sw : 0);
    // two items per workgroup when both products share the launch (a dX item and dW tiles interleave well), one when a
    // product runs alone (half the split-K partials: measured 37 instead of 47 us for dX of the 4096x4096 layer)
    int64_t len = all / (want_dx && want_dw ? 512 : 256);
    if (len < 8) len = 8;
    const bool alone = want_dx != want_dw;
    auto split = [len, kt, alone](int64_t steps, FcPlan &pl) {
        int64_t n = (steps + len / 2) / len;
        // a product that runs alone: at most one item per workgroup (256 of them), so that no workgroup takes a second
        // item while the others idle (8 tiles x 33 splits = 264 items ran as two rounds)
        if (alone && pl.tiles <= 256 && n * pl.tiles > 256) n = 256 / pl.tiles;
        if (n < 1) n = 1;
        const int64_t per = (steps + n - 1) / n;
        pl.k_per_split = (int)(per * kt);
        pl.n_split = (int)((steps + per - 1) / per);
        pl.partial_bytes = pl.n_split > 1 ? (size_t)pl.tiles * pl.n_split * FC2_TM * FC2_TN * sizeof(float) : 0;
    };
    split(sx, dx); split(sw, dw);
}

// The two products on two groups of workgroups (FcPairArgs::gx) where that needs fewer split-K partials than the common
// list for the same longest workgroup: group sizes in proportion to the products' K steps (multiples of 8: every XCD
// gets its share of both), a split product cut into about one item per workgroup of its group.  Returns gx, or 0 to keep
// the common list; dx and dw are replaced by the group plan when it is taken.
int fc2_group_plan(int64_t B, int64_t in, int64_t out, FcPlan &dx, FcPlan &dw, int kt = FC2_KT)
{
    const int G = 256;
    const int64_t sx = (out + kt - 1) / kt, sw = (B + kt - 1) / kt;
    const int64_t all_x = dx.tiles * sx, all_w = dw.tiles * sw;
    if (dx.tiles * dx.n_split + dw.tiles * dw.n_split < G) return 0;
    int gx = (int)((G * all_x + (all_x + all_w) / 2) / (all_x + all_w) + 4) / 8 * 8;
    gx = gx < 8 ? 8 : gx > G - 8 ? G - 8 : gx;
    auto cut = [kt](int64_t steps, FcPlan pl, int g) {
        int64_t n = pl.tiles >= g ? 1 : g / pl.tiles;
        const int64_t most = steps / 8 > 0 ? steps / 8 : 1;            // at least eight K steps per item
        if (n > most) n = most;
        const int64_t per = (steps + n - 1) / n;
        pl.k_per_split = (int)(per * kt);
        pl.n_split = (int)((steps + per - 1) / per);
        pl.partial_bytes = pl.n_split > 1 ? (size_t)pl.tiles * pl.n_split * FC2_TM * FC2_TN * sizeof(float) : 0;
        return pl;
    };
    const FcPlan gdx = cut(sx, dx, gx), gdw = cut(sw, dw, G - gx);
    auto rounds = [](const FcPlan &pl, int g) { return (pl.tiles * pl.n_split + g - 1) / g * (int64_t)(pl.k_per_split); };
    const int64_t longest_groups = rounds(gdx, gx) > rounds(gdw, G - gx) ? rounds(gdx, gx) : rounds(gdw, G - gx);
    // the common list: workgroup w takes items p*G + (w or G-1-w) of the concatenated lists
    const int64_t n0 = dx.tiles * dx.n_split, total = n0 + dw.tiles * dw.n_split;
    int64_t longest_common = 0;
    for (int w = 0; w < G; ++w) {
        int64_t len = 0;
        for (int64_t ps = 0; ps * G < total; ++ps) {
            const int64_t t = ps * G + ((ps & 1) ? G - 1 - w : w);
            if (t < total) len += t < n0 ? dx.k_per_split : dw.k_per_split;
        }
        if (len > longest_common) longest_common = len;
    }
    if (longest_groups > longest_common || gdx.partial_bytes + gdw.partial_bytes >= dx.partial_bytes + dw.partial_bytes) return 0;
    if ((gdx.tiles * gdx.n_split + gx - 1) / gx > FC2_MAX_ITEMS || (gdw.tiles * gdw.n_split + G - gx - 1) / (G - gx) > FC2_MAX_ITEMS) return 0;
    dx = gdx; dw = gdw;
    return gx;
}

// ---- fully connected layers straight from global memory (fc_direct_kernel.h) ----------------------------------
struct FcdPlan { int mf, kw, n_split, steps_per_split, tiles_m, tiles, groups; size_t partial_bytes; float us; };

// Shape of one product on fc_direct_kernel, by modelled time: 32 or 64 rows a wavefront, the wavefronts that share a tile's
// reduction, and (where that leaves most of `room` CUs idle and the partials fit `cap` bytes) splits over workgroups.
// Calibrated on layers from 16x64x64 to 512x2048x2048: a step of a wavefront takes about 0.45 us (0.55 with 64 rows), twice that
// where the dense operand comes from HBM; adding up through LDS about 0.5 us a halving; a second launch 5 us, and from 32 splits on
// 0.8 for every eight more that it adds (a latency each: dX of 32x64x8192 in 128 splits 24 us, in 16 splits of eight wavefronts 14); so one, as many as fit, or 16 in between.
FcdPlan fcd_plan(int64_t M, int64_t N, int64_t K, bool i8, int room, size_t cap)
{
    FcdPlan best{};
    best.us = -1.0f;
    const int steps = (int)((K + (i8 ? 31 : 15)) / (i8 ? 32 : 16));
    const int64_t tn = (N + fcd_tn(i8) - 1) / fcd_tn(i8);
    const float cold = (float)K * N * (i8 ? 1.0f : 4.0f) > 32.0e6f ? 2.0f : 1.0f;
    for (int mf = 1; mf <= (i8 ? 1 : 2); ++mf) {
        const int64_t tm = (M + 32 * mf - 1) / (32 * mf), tiles = tm * tn;
        const float step = cold * (mf == 2 ? 0.55f : 0.45f);
        for (int kw = 1, halvings = 0; kw <= FCD_WAVES && kw <= steps; kw *= 2, ++halvings) {
            const int64_t groups = (tiles * kw + FCD_WAVES - 1) / FCD_WAVES;
            int most = steps / (4 * kw);
            if (most > room / groups) most = (int)(room / groups);
            if (most > 1 && (size_t)most * M * N * 4 > cap) most = (int)(cap / ((size_t)M * N * 4));
            for (int n = 1;; n = n == 1 && most > 32 ? 16 : most) {
                const int per = (steps + n - 1) / n, ns = (steps + per - 1) / per;
                const float rounds = groups * ns <= room ? 1.0f : (float)(groups * ns) / room;
                float us = rounds * (1.5f + (float)((per + kw - 1) / kw) * step + 0.5f * halvings);
                if (ns > 1) us += 5.0f + (ns > 32 ? 0.8f * (float)((ns - 25) / 8) : 0.0f) + (float)ns * M * N * 8.0f / 4.0e6f;
                if (best.us < 0.0f || us < best.us)
                    best = FcdPlan{mf, kw, ns, per, (int)tm, (int)tiles, (int)groups, ns > 1 ? (size_t)ns * M * N * 4 : 0, us};
                if (n >= most) break;
            }
        }
    }
    return best;
}

// What the kernel takes: rows of at least NF (MF) elements, 32-bit offsets.
bool fcd_ok(bool kfast, int64_t M, int64_t N, int64_t K, int64_t lda, bool i8)
{
    return N >= (i8 ? 4 : 2) && (kfast || M >= 2) && M * N >= 4 && lda < (1 << 24) && N < (1 << 24) && (!kfast || M * lda < ((int64_t)1 << 31)) && K >= 1 &&
           M < ((int64_t)1 << 24) && K < ((int64_t)1 << 24);
}

// The products of `a` that are asked for, on the direct kernel, with the quantiser's pending sums beside them.
hipError_t launch_fc_direct(const LinearArgs &a, bool want_dx, bool want_dw, const StatsJob &job, hipStream_t s)
{
    static bool raised = false;                                      // with its static LDS above 64 KiB: allowed per kernel, once
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&fc_direct_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 64 << 10);
        if (e != hipSuccess) return e;
        raised = true;
    }
    FcdArgs fa{};
    char *scratch = (char *)a.scratch;
    // the chip in proportion to the products' multiply-adds, which are the same: half each
    const int room = want_dx && want_dw ? 128 : 256;
    size_t left = a.scratch_bytes & ~(size_t)255, lds = 0;
    int blocks = 0, reduce[2] = {0, 0};
    auto fill = [&](int which, bool kfast, bool i8, const void *Bop, int64_t M, int64_t K, void *out) {
        const FcdPlan pl = fcd_plan(M, a.in, K, i8, room, left);
        FcdProblem &p = fa.prob[which];
        p.A = a.codes; p.lda = a.out; p.B = Bop; p.ldb = a.in; p.out = out; p.partial = scratch;
        p.M = (int)M; p.N = (int)a.in; p.K = (int)K;
        p.tiles_m = pl.tiles_m; p.tiles = pl.tiles; p.kw = pl.kw; p.n_split = pl.n_split; p.steps_per_split = pl.steps_per_split;
        p.groups = pl.groups; p.form = fcd_form(i8, kfast, pl.mf); p.scale = i8 ? Scale{1.0f, nullptr} : Scale{a.step, a.step_dev};
        const size_t used = align_up(pl.partial_bytes, 256);
        scratch += used; left = left > used ? left - used : 0;
        blocks += pl.groups * pl.n_split;
        if (pl.n_split > 1) reduce[which] = (int)((M * a.in + 1023) / 1024);
        const size_t slots = pl.kw > 1 ? (size_t)(FCD_WAVES / 2) * pl.mf * fcd_tn(i8) * 32 * 4 : 0;
        if (slots > lds) lds = slots;
    };
    if (want_dx) fill(0, true, a.W8 != nullptr, a.W8 ? (const void *)a.W8 : (const void *)a.W, a.B, a.out, a.dX);
    fa.first1 = blocks;
    if (want_dw) fill(1, false, a.x_dtype == DBP_I8, a.X, a.out, a.B, a.dW);
    fa.stats = job; fa.gate = a.gate;
    if (a.fused) {
        const hipError_t e = launch_fc_fused(fa, *a.fused, blocks + 1, lds, s);
        if (e != hipSuccess) return e;
    } else {
        hipLaunchKernelGGL(fc_direct_kernel, dim3((unsigned)(blocks + job.workgroups())), dim3(64 * FCD_WAVES), lds, s, fa);
    }
    if (reduce[0] + reduce[1] > 0)
        hipLaunchKernelGGL(fcd_reduce_kernel, dim3((unsigned)(reduce[0] + reduce[1])), dim3(256), 0, s, fa, reduce[0]);
    return hipGetLastError();
}

FcProblem fc_problem(bool a_kfast, const int8_t *A, int64_t lda, const float *B, int64_t ldb, int M, int N, int K,
                     Scale scale, float *out, const FcPlan &pl, char *&scratch)
{
    FcProblem p;
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb; p.out = out; p.ldc = N;
    p.M = M; p.N = N; p.K = K; p.scale = scale; p.a_kfast = a_kfast ? 1 : 0;
    p.tiles_m = pl.tiles_m; p.n_split = pl.n_split; p.k_per_split = pl.k_per_split;
    p.n_items = (int)(pl.tiles * pl.n_split);
    p.partial = (float *)scratch;
    p.nt_pq = 0; p.nt_spi = 1; p.nt_a_img = 0; p.nt_b_img = 0;
    scratch += align_up(pl.partial_bytes, 256);
    return p;
}

}  // namespace

size_t linear_scratch_bytes(int64_t B, int64_t in, int64_t out)
{
    // generic kernel: split-K partials of the larger of the two products, at the split the launcher would choose
    auto part = [](int64_t M, int64_t N, int64_t K) {
        int64_t tiles = ((M + TM - 1) / TM) * ((N + TN - 1) / TN);
        Split sp = choose_split(tiles, K, 16);          // smallest K step (fp32 mode) gives the largest split
        return sp.n > 1 ? (size_t)sp.n * M * N * 4 : (size_t)0;
    };
    size_t a = part(B, in, out), b = part(out, in, B);
    const size_t generic = align_up(a > b ? a : b, 256);
    // staged kernels: both products in one launch, each with its own partials (the direct kernel makes do with what there is)
    size_t fast = 0;
    for (int m = 1; m < 4; ++m) {                               // every combination of products a call can ask for
        FcPlan dx2, dw2;
        for (int kt = FC2_KT; kt <= FC2I_KT; kt *= 2) {              // the bf16 kernel's K step and the int8 kernel's
            fc2_plans(B, in, out, (m & 1) != 0, (m & 2) != 0, dx2, dw2, kt);
            const size_t fast2 = ((m & 1) ? align_up(dx2.partial_bytes, 256) : 0) + ((m & 2) ? align_up(dw2.partial_bytes, 256) : 0);
            if (fast2 > fast) fast = fast2;
        }
    }
    const size_t gather = align_up(linear_gather_scratch_bytes(B, in, out), 256);      // split partials of the gather dX kernel
    const size_t mfma = generic > fast ? generic : fast;
    return (mfma > gather ? mfma : gather) + 256;
}

// dW of a 1x1, stride-1, unpadded convolution: dW[k][c] = sum_n sum_p code[n][k][p] X[n][c][p] is the batched,
// reduction-contiguous form of the FC kernels (fc2_kernel.h / fc2_i8_kernel.h, NT) straight on the NCHW tensors: no copy
// pass.  kt = reduction indices per K step of the kernel (32 with fp32 activations, 64 with int8 activations).
struct Conv1x1Plan { bool ok; int n_split, imgs_per_split, spi, tiles_m, tiles_n, kt; size_t partial_bytes; float us; };

Conv1x1Plan conv1x1_dw_plan(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t pad, int64_t stride,
                            int kt = FC2_KT)
{
    Conv1x1Plan pl;
    pl.ok = false; pl.partial_bytes = 0;
    const int64_t PQ = H * Wd;
    if (!(R == 1 && S == 1 && pad == 0 && stride == 1)) return pl;
    pl.kt = kt;
    if (K < FC2_TM / 4 || C < 4 || PQ < kt) return pl;              // row tiles at least a quarter full; whole windows
    if (C * PQ >= ((int64_t)1 << 29) || K * PQ >= ((int64_t)1 << 31) || K * C >= ((int64_t)1 << 30)) return pl;   // 32-bit lane offsets
    pl.spi = (int)((PQ + kt - 1) / kt);
    if (N * pl.spi >= ((int64_t)1 << 25)) return pl;                              // the reduction axis counts windows of kt
    pl.tiles_m = (int)((K + FC2_TM - 1) / FC2_TM); pl.tiles_n = (int)((C + FC2_TN - 1) / FC2_TN);
    const int64_t tiles = (int64_t)pl.tiles_m * pl.tiles_n;
    int64_t n = tiles >= 256 ? 1 : 256 / tiles;                                   // at most one item per workgroup
    if (n > N) n = N;
    while (n > 1 && ((N + n - 1) / n) * pl.spi < 8) --n;                          // at least eight steps per item
    pl.imgs_per_split = (int)((N + n - 1) / n);
    pl.n_split = (int)((N + pl.imgs_per_split - 1) / pl.imgs_per_split);
    if (tiles * pl.n_split > (int64_t)FC2_MAX_ITEMS * 256) return pl;
    pl.partial_bytes = pl.n_split > 1 ? (size_t)tiles * pl.n_split * FC2_TM * FC2_TN * sizeof(float) : 0;
    // a step takes 0.8 us (int8: 0.5), more when all CUs stream from HBM; 12 to 14 us for the ends and the partial sums
    const float wgs = tiles * pl.n_split < 256 ? (float)(tiles * pl.n_split) / 256.0f : 1.0f, rounds = (float)((tiles * pl.n_split + 255) / 256);
    pl.us = (kt == FC2_KT ? 14.0f : 12.0f) + rounds * pl.imgs_per_split * pl.spi * (kt == FC2_KT ? 0.8f + 0.5f * wgs : 0.5f + 0.6f * wgs);
    pl.ok = true;
    return pl;
}

template <bool I8>
hipError_t launch_conv1x1_dw(const ConvArgs &a, const Conv1x1Plan &pl, const int8_t *codes, Scale scale, char *scratch, hipStream_t s)
{
    static bool raised = false;
    if (!raised) {
        hipError_t e = I8 ? hipFuncSetAttribute(reinterpret_cast<const void *>(&fc2_i8_pair_kernel<true>),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, FC2I_LDS_BYTES)
                          : hipFuncSetAttribute(reinterpret_cast<const void *>(&fc2_pair_kernel<true, 3>),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, FC2_LDS_BYTES);
        if (e != hipSuccess) return e;
        if (!I8) e = hipFuncSetAttribute(reinterpret_cast<const void *>(&fc2_pair_kernel<true, 2>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, FC2_LDS_BYTES);
        if (e != hipSuccess) return e;
        raised = true;
    }
    const int64_t PQ = a.H * a.Wd;
    FcPairArgs pa;
    FcProblem &p = pa.prob[0];
    p.A = codes; p.lda = PQ; p.B = (const float *)a.X; p.ldb = PQ; p.out = (float *)a.dW; p.ldc = a.C;
    p.partial = (float *)scratch;
    p.M = (int)a.K; p.N = (int)a.C; p.K = (int)(a.N * pl.spi * pl.kt);
    p.k_per_split = pl.imgs_per_split * pl.spi * pl.kt; p.n_split = pl.n_split; p.tiles_m = pl.tiles_m;
    p.n_items = pl.tiles_m * pl.tiles_n * pl.n_split;
    p.scale = scale; p.a_kfast = 1;
    p.nt_pq = (int)PQ; p.nt_spi = pl.spi; p.nt_a_img = a.kt() * PQ; p.nt_b_img = a.ct() * PQ;
    pa.prob[1] = p;
    pa.prob[1].n_items = 0;
    pa.stats = StatsJob{nullptr, 0, nullptr, nullptr, 0, nullptr, 0.0f, nullptr};
    pa.gate = a.gate;
    const int grid = p.n_items < 256 ? p.n_items : 256;
    if constexpr (I8) hipLaunchKernelGGL(fc2_i8_pair_kernel<true>, dim3(grid), dim3(512), FC2I_LDS_BYTES, s, pa);
    else if (a.two_planes) hipLaunchKernelGGL((fc2_pair_kernel<true, 2>), dim3(grid), dim3(512), FC2_LDS_BYTES, s, pa);
    else              hipLaunchKernelGGL((fc2_pair_kernel<true, 3>), dim3(grid), dim3(512), FC2_LDS_BYTES, s, pa);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (pl.n_split > 1) {
        const int tiles = pl.tiles_m * pl.tiles_n;
        if constexpr (I8) hipLaunchKernelGGL(fc2_i8_reduce_kernel, dim3(32 * tiles), dim3(256), 0, s, pa, tiles);
        else              hipLaunchKernelGGL(fc2_reduce_kernel, dim3(32 * tiles), dim3(256), 0, s, pa, tiles);
        e = hipGetLastError();
    }
    return e;
}

size_t conv_scratch_bytes(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t pad, int64_t stride)
{
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1;
    auto part = [](int64_t M, int64_t Nn, int64_t Kr, int64_t gran) {
        int64_t tiles = ((M + TM - 1) / TM) * ((Nn + TN - 1) / TN);
        Split sp = choose_split(tiles, Kr, (int)gran);
        return sp.n > 1 ? (size_t)sp.n * M * Nn * 4 : (size_t)0;
    };
    size_t dx = part(N * H * Wd, C, R * S * ((K + 7) / 8 * 8), 16);
    const int64_t PQp16 = (P * Q + 15) / 16 * 16;
    size_t dw = part(K, C * R * S, N * PQp16, 16);
    size_t big = dx > dw ? dx : dw;
    for (int i8 = 0; i8 < 2; ++i8) {
        const ConvDwPlan pl = conv_dw_plan(N, C, H, Wd, K, R, S, pad, i8 != 0);
        if (pl.ok && pl.partial_bytes > big) big = pl.partial_bytes;
    }
    const ConvDwI8Plan p8 = conv_dw_i8_plan(N, C, H, Wd, K, R, S, pad);
    if (p8.ok && p8.partial_bytes > big) big = p8.partial_bytes;
    for (int i8 = 0; i8 < 2; ++i8) {
        const Conv1x1Plan p1 = conv1x1_dw_plan(N, C, H, Wd, K, R, S, pad, stride, i8 ? FC2I_KT : FC2_KT);
        if (p1.ok && p1.partial_bytes > big) big = p1.partial_bytes;
    }
    for (int i8 = 0; i8 < 2; ++i8)
        for (int planes = i8 ? 3 : 2; planes <= 3; ++planes) {
            const ConvDwtPlan pd = conv_dwt_plan(N, C, H, Wd, K, R, S, pad, stride, i8 != 0, planes);
            if (pd.ok && pd.partial_bytes > big) big = pd.partial_bytes;
        }
    const size_t padded = (size_t)(N * K * ((P * Q + 3) / 4 * 4));    // dX: the codes in planes that start on 4-byte boundaries
    if (padded > big) big = padded;
    return relayout_bytes(K, C, R, S) + align_up(big, 256) + 256;
}

// Which kernel computes each product of a fully connected layer (the same for a launch and for dbp_plan_linear).
struct FcChoice { bool dx_staged, dw_staged, dx_direct, dw_direct; };

static FcChoice linear_choose(const LinearArgs &a)
{
    const int64_t B = a.B, in = a.in, out = a.out;
    const bool dx_i8 = a.W8 != nullptr, dw_i8 = a.x_dtype == DBP_I8;
    // What the staged kernels take: a full window of reduction indices, runs of 16 rows in dW, 32-bit lane offsets ...
    const bool small_index = B * in < (1ll << 30) && out * in < (1ll << 30) && B * out < (1ll << 30);
    const bool can_dx = a.dX && small_index && out >= (dx_i8 ? FC2I_KT : FC2_KT) && in >= (dx_i8 ? 8 : 4);
    const bool can_dw = a.dW && small_index && B >= (dw_i8 ? FC2I_KT : FC2_KT) && out >= 16 && in >= (dw_i8 ? 8 : 4);
    // ... and what they are the faster ones for, by multiply-adds of a product.  Two planes exist on the staged kernel only.
    const double macs = (double)B * in * out;
    const bool short_dx = B <= FC2_TM / 2, short_dw = out <= FC2_TM / 2, two = a.two_planes && !dx_i8;   // rows for half a tile at most
    FcChoice c{};
    if (a.dX && a.dW && dx_i8 == dw_i8) {
        if (!short_dx && !short_dw) {
            // one launch for both.  Direct / staged (us): 256x1024x1024 15 / 19, 160x2048x2048 29 / 24, 256x1024x4096 35 / 24
            c.dx_staged = c.dw_staged = can_dx && can_dw && (macs > 3.0e8 || two);
        } else if (macs > (dx_i8 ? 5.0e9 : 1.65e9)) {
            // A product of few rows wastes most of its tiles, but the direct kernel cuts the dense operand again for every 32 or 64 rows.  Both
            // direct / dX direct, dW staged / both staged (us): 32x8192x8192 146 / 105 / 141, 96x8192x8192 261 / 153 / 162, 128x8192x8192 281 / 160 / 160,
            // 128x4096x4096 56 / 58 / 49, 64x4096x4096 43 / 44 / 56; with the rows in dX 4096x8192x100 116 / 113 / 82; int8 96x4096x16384 132 / 96 / 94, 128x8192x4096 49 / - / 54
            c.dx_staged = can_dx && B > 96;
            c.dw_staged = can_dw && out > 96;
        }
    } else {
        // A product alone, or two kinds of product (a launch each).  Direct / staged (us): dX 160x1024x4096 22 / 25, 256x2048x2048 26 / 24. Alone: dX with few
        // steps of reduction 512x8192x64 13 / 11; dW of many tiles 64x2048x2048 13 / 11, 59x2217x1811 14 / 11 (of few tiles 379x112x3790 16 / 26)
        const bool alone = !a.dX || !a.dW;
        c.dx_staged = can_dx && !short_dx && (macs > 3.0e8 || two || (alone && !dx_i8 && short_dw && macs > 2.0e8));
        c.dw_staged = can_dw && !short_dw && (macs > 3.0e8 || two || (alone && !dw_i8 && (double)in * out > 1.5e6 && macs > 1.5e8));
    }
    for (int i8 = 0; i8 < 2; ++i8) {                                      // the per-workgroup item table is fixed
        const bool dx_here = c.dx_staged && dx_i8 == (i8 != 0), dw_here = c.dw_staged && dw_i8 == (i8 != 0);
        FcPlan pdx, pdw;
        if (dx_here || dw_here) fc2_plans(B, in, out, dx_here, dw_here, pdx, pdw, i8 ? FC2I_KT : FC2_KT);
        if ((dx_here ? pdx.tiles * pdx.n_split : 0) + (dw_here ? pdw.tiles * pdw.n_split : 0) > (int64_t)FC2_MAX_ITEMS * 256) {
            if (dx_here) c.dx_staged = false;
            if (dw_here) c.dw_staged = false;
        }
    }
    c.dx_direct = a.dX && !c.dx_staged && fcd_ok(true, B, in, out, out, dx_i8);
    c.dw_direct = a.dW && !c.dw_staged && fcd_ok(false, out, in, B, out, dw_i8);
    return c;
}

// Few gradients: every workgroup of the direct kernel quantises all of them for itself, which is a launch less (of two; of three with the step size), and one
// more workgroup writes what the quantiser leaves.  8192 gradients are sixteen a thread.  Launches of their own / one launch (us): 8192 gradients 64x784x128 12.1 / 9.1,
// 16x8192x512 15.1 / 13.5, with the step size 64x784x128 17.4 / 14.8; of 16384 and more (forty a thread allowed) 64x784x256 12.3 / 11.4, with the step
// size 17.9 / 18.2, 16x1024x1000 14.5 / 14.8, 64x784x300 12.4 / 12.6, 40x4096x500 14.5 / 21.5.
// Workgroups beyond the first round over the chip quantise once more behind the others, and what a launch less saves is soon gone, the sooner the more
// gradients there are and the more a workgroup does with them.  The lines below, with the workgroups of the products, launches of their own / one launch (us):
//   with the step size  52x8069x106 254 18.1 / 14.2, 16x8192x500 256 21.5 / 26.2, 64x16384x96 256 21.5 / 24.1, 512x16384x16 384 32.1 / 36.0, 512x262144x16 4608 291 / 419
//   ... to 4096         128x65536x32 384 32.0 / 27.6, 128x131072x32 768 46.9 / 44.0, 5x83989x367 1151 52.9 / 55.1
//   int8 weights        64x65536x96 320 17.0 / 16.9, 378x30130x20 472 23.4 / 22.9, 64x131072x96 640 24.2 / 26.2; to 4096: 183x89604x21 614 28.9 / 25.5, 9x56482x389 830 26.8 / 27.6
//   neither             16x65536x500 1152 59.1 / 55.3, 3x19865x2486 1673 120.9 / 119.5, 16x131072x500 2304 145 / 149; int8 activations 64x146865x123 861 41.8 / 43.4;
//                       to 6144: 64x262144x96 1536 98.1 / 89.7
static int64_t fcd_workgroups(const LinearArgs &a)                    // of both products, as launch_fc_direct plans them
{
    const int room = a.dX && a.dW ? 128 : 256;
    size_t left = a.scratch_bytes & ~(size_t)255;
    int64_t n = 0;
    if (a.dX) {
        const FcdPlan pl = fcd_plan(a.B, a.in, a.out, a.W8 != nullptr, room, left);
        const size_t used = align_up(pl.partial_bytes, 256);
        left = left > used ? left - used : 0;
        n += (int64_t)pl.groups * pl.n_split;
    }
    if (a.dW) {
        const FcdPlan pl = fcd_plan(a.out, a.in, a.B, a.x_dtype == DBP_I8, room, left);
        n += (int64_t)pl.groups * pl.n_split;
    }
    return n;
}

bool linear_fused_ok(const LinearArgs &a, bool layer)
{
    const int64_t n = a.B * a.out;
    if (!a.codes || n > kFusedMax || (!a.dX && !a.dW) || a.gate.flag) return false;
    const FcChoice c = linear_choose(a);
    if ((a.dX && !c.dx_direct) || (a.dW && !c.dw_direct)) return false;
    const int64_t most = layer ? (n > 4096 ? 255 : 1024) : a.W8 ? (n > 4096 ? 512 : 768) : n > 6144 ? (a.x_dtype == DBP_I8 ? 768 : 2000) : 8192;
    // (a plan has no more workgroups than its room or its tiles of 32 rows: small layers are spared the planning, 0.3 us of a call's 9)
    const int64_t room = a.dX && a.dW ? 128 : 256;
    auto bound = [&](int64_t M, bool i8) { const int64_t tiles = (M + 31) / 32 * ((a.in + fcd_tn(i8) - 1) / fcd_tn(i8)); return tiles > room ? tiles : room; };
    if ((a.dX ? bound(a.B, a.W8 != nullptr) : 0) + (a.dW ? bound(a.out, a.x_dtype == DBP_I8) : 0) <= most) return true;
    return fcd_workgroups(a) <= most;
}

// ------------------------------------------------------------------------------------------------
// Fully connected layer.  dX = q.W : rows b, cols i, reduction o.   dW = q^T.X : rows o, cols i, reduction b.
// ------------------------------------------------------------------------------------------------
hipError_t launch_linear_mfma(const LinearArgs &a, hipStream_t s)
{
    const int B = (int)a.B, in = (int)a.in, out = (int)a.out;
    hipError_t e = hipSuccess;
    RowMajorOut om{a.in};
    StatsJob pending = a.stats_job;
    if (a.plan_only && (!a.codes || a.W8)) { *a.plan_only = 1; return hipSuccess; }
    if (a.codes) {
        const bool dx_i8 = a.W8 != nullptr, dw_i8 = a.x_dtype == DBP_I8;
        const FcChoice c = linear_choose(a);
        if (a.plan_only) {
            // gated: both requested products on kernels that take a gate, fp32 operands
            if ((a.dX && !c.dx_staged && !c.dx_direct) || (a.dW && (dw_i8 || (!c.dw_staged && !c.dw_direct)))) *a.plan_only = 1;
            return hipSuccess;
        }
        // staged products of one kind share a launch
        for (int i8 = 0; i8 < 2; ++i8) {
            const bool dx_here = c.dx_staged && dx_i8 == (i8 != 0), dw_here = c.dw_staged && dw_i8 == (i8 != 0);
            if (!dx_here && !dw_here) continue;
            const int kt = i8 ? FC2I_KT : FC2_KT;
            FcPlan pdx, pdw;
            fc2_plans(B, in, out, dx_here, dw_here, pdx, pdw, kt);
            const int gx = dx_here && dw_here ? fc2_group_plan(B, in, out, pdx, pdw, kt) : 0;
            static bool raised = false;
            if (!raised) {
                const void *fns[3] = {reinterpret_cast<const void *>(&fc2_pair_kernel<false, 3>), reinterpret_cast<const void *>(&fc2_pair_kernel<false, 2>),
                                      reinterpret_cast<const void *>(&fc2_i8_pair_kernel<false>)};
                for (int f = 0; f < 3; ++f) {
                    e = hipFuncSetAttribute(fns[f], hipFuncAttributeMaxDynamicSharedMemorySize, f == 2 ? FC2I_LDS_BYTES : FC2_LDS_BYTES);
                    if (e != hipSuccess) return e;
                }
                raised = true;
            }
            char *scratch = (char *)a.scratch;
            const Scale scale = i8 ? Scale{1.0f, nullptr} : Scale{a.step, a.step_dev};
            FcPairArgs pa;
            if (!dx_here) { pdx.n_split = 1; pdx.partial_bytes = 0; }
            if (!dw_here) { pdw.n_split = 1; pdw.partial_bytes = 0; }
            pa.prob[0] = fc_problem(true, a.codes, a.out, dx_i8 ? (const float *)a.W8 : a.W, a.in, B, in, out, scale, a.dX, pdx, scratch);
            pa.prob[1] = fc_problem(false, a.codes, a.out, (const float *)a.X, a.in, out, in, B, scale, (float *)a.dW, pdw, scratch);
            if (!dx_here) pa.prob[0].n_items = 0;
            if (!dw_here) pa.prob[1].n_items = 0;
            if ((size_t)(scratch - (char *)a.scratch) > a.scratch_bytes) return hipErrorInvalidValue;
            pa.stats = pending;                                // finished by a stager wavefront of the last workgroup
            pending = StatsJob{};
            pa.gx = gx; pa.gate = a.gate;
            const int total = pa.prob[0].n_items + pa.prob[1].n_items;
            const int grid = total < 256 ? total : 256;        // persistent: one workgroup per CU (256 whenever gx > 0)
            if (i8)                hipLaunchKernelGGL(fc2_i8_pair_kernel<false>, dim3(grid), dim3(512), FC2I_LDS_BYTES, s, pa);
            else if (a.two_planes) hipLaunchKernelGGL((fc2_pair_kernel<false, 2>), dim3(grid), dim3(512), FC2_LDS_BYTES, s, pa);
            else                   hipLaunchKernelGGL((fc2_pair_kernel<false, 3>), dim3(grid), dim3(512), FC2_LDS_BYTES, s, pa);
            const int tiles0 = dx_here && pdx.n_split > 1 ? (int)pdx.tiles : 0, tiles1 = dw_here && pdw.n_split > 1 ? (int)pdw.tiles : 0;
            if (tiles0 + tiles1 > 0) {
                if (i8) hipLaunchKernelGGL(fc2_i8_reduce_kernel, dim3(32 * (tiles0 + tiles1)), dim3(256), 0, s, pa, tiles0);
                else    hipLaunchKernelGGL(fc2_reduce_kernel, dim3(32 * (tiles0 + tiles1)), dim3(256), 0, s, pa, tiles0);
            }
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        // the rest in one launch of the direct kernel, or (rows shorter than its vectors) product by product on the generic one
        if (c.dx_direct || c.dw_direct) {
            e = launch_fc_direct(a, c.dx_direct, c.dw_direct, pending, s);
            if (e != hipSuccess) return e;
            pending = StatsJob{};
        }
        if (pending.n || pending.bias_len) { e = launch_stats_job(pending, s); if (e != hipSuccess) return e; }
        if (a.dX && !c.dx_staged && !c.dx_direct) {
            if (dx_i8) {
                MatrixLoader<MODE_I8, true, true>   al{a.codes, a.out, B, out};
                MatrixLoader<MODE_I8, false, false> bl{a.W8, a.in, in, out};
                e = run_gemm<MODE_I8>(al, bl, om, B, in, out, k_step<MODE_I8>(), Scale{1.0f, nullptr}, (int32_t *)a.dX, a.scratch, a.scratch_bytes, s);
            } else {
                MatrixLoader<MODE_BF16, true, true>   al{a.codes, a.out, B, out};
                MatrixLoader<MODE_BF16, false, false> bl{a.W, a.in, in, out};
                e = run_gemm<MODE_BF16>(al, bl, om, B, in, out, k_step<MODE_BF16>(), Scale{a.step, a.step_dev}, a.dX, a.scratch, a.scratch_bytes, s);
            }
            if (e != hipSuccess) return e;
        }
        if (a.dW && !c.dw_staged && !c.dw_direct) {
            if (dw_i8) {
                MatrixLoader<MODE_I8, true, false>  al{a.codes, a.out, out, B};
                MatrixLoader<MODE_I8, false, false> bl{(const int8_t *)a.X, a.in, in, B};
                e = run_gemm<MODE_I8>(al, bl, om, out, in, B, k_step<MODE_I8>(), Scale{1.0f, nullptr}, (int32_t *)a.dW, a.scratch, a.scratch_bytes, s);
            } else {
                MatrixLoader<MODE_BF16, true, false>  al{a.codes, a.out, out, B};
                MatrixLoader<MODE_BF16, false, false> bl{(const float *)a.X, a.in, in, B};
                e = run_gemm<MODE_BF16>(al, bl, om, out, in, B, k_step<MODE_BF16>(), Scale{a.step, a.step_dev}, (float *)a.dW, a.scratch, a.scratch_bytes, s);
            }
        }
        return e;
    }
    // dense baseline
    if (pending.n || pending.bias_len) { e = launch_stats_job(pending, s); if (e != hipSuccess) return e; }
    if (a.dX) {
        MatrixLoader<MODE_F32, false, true>  al{(const float *)a.dense, a.out, B, out};
        MatrixLoader<MODE_F32, false, false> bl{a.W, a.in, in, out};
        e = run_gemm<MODE_F32>(al, bl, om, B, in, out, k_step<MODE_F32>(), Scale{1.0f, nullptr}, a.dX, a.scratch, a.scratch_bytes, s);
        if (e != hipSuccess) return e;
    }
    if (a.dW && a.x_dtype == DBP_F32) {
        MatrixLoader<MODE_F32, false, false> al{(const float *)a.dense, a.out, out, B};
        MatrixLoader<MODE_F32, false, false> bl{(const float *)a.X, a.in, in, B};
        e = run_gemm<MODE_F32>(al, bl, om, out, in, B, k_step<MODE_F32>(), Scale{1.0f, nullptr}, (float *)a.dW, a.scratch, a.scratch_bytes, s);
    } else if (a.dW) {
        MatrixLoader<MODE_I8, false, false> al{(const int8_t *)a.dense, a.out, out, B};
        MatrixLoader<MODE_I8, false, false> bl{(const int8_t *)a.X, a.in, in, B};
        e = run_gemm<MODE_I8>(al, bl, om, out, in, B, k_step<MODE_I8>(), Scale{1.0f, nullptr}, (int32_t *)a.dW, a.scratch, a.scratch_bytes, s);
    }
    return e;
}

// Clears n 4-byte words (the output pixels of a strided layer that no tap reaches).
__global__ __launch_bounds__(256) void zero_words_kernel(uint32_t *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0u;
}

// Grouped convolution with few channels per group, run as ONE ungrouped layer: the weights [K][Cg][RS] are expanded into
// the block-diagonal [K][C][RS] (zero outside a channel's own group: those products add exact zeros), and the diagonal
// blocks of the ungrouped dW are copied back.  4-byte elements either way (fp32 weights; fp32 or int32 dW).
__global__ __launch_bounds__(256) void group_weights_expand_kernel(const uint32_t *W, uint32_t *full, int K, int C, int Cg, int Kg, int RS)
{
    const int64_t total = (int64_t)K * C * RS;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int rs = (int)(i % RS);
        const int64_t kc = i / RS;
        const int c = (int)(kc % C), k = (int)(kc / C);
        const bool own = c / Cg == k / Kg;
        full[i] = own ? W[((int64_t)k * Cg + c % Cg) * RS + rs] : 0u;
    }
}

__global__ __launch_bounds__(256) void group_dw_extract_kernel(const uint32_t *full, uint32_t *dW, int K, int C, int Cg, int Kg, int RS)
{
    const int64_t total = (int64_t)K * Cg * RS;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int rs = (int)(i % RS);
        const int64_t kc = i / RS;
        const int cl = (int)(kc % Cg), k = (int)(kc / Cg);
        dW[i] = full[((int64_t)k * C + (k / Kg) * Cg + cl) * RS + rs];
    }
}

hipError_t launch_group_weights_expand(const float *W, float *full, int64_t K, int64_t C, int64_t groups, int64_t RS, hipStream_t s)
{
    const int64_t total = K * C * RS;
    const int blocks = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
    hipLaunchKernelGGL(group_weights_expand_kernel, dim3(blocks), dim3(256), 0, s, (const uint32_t *)W, (uint32_t *)full, (int)K, (int)C,
                       (int)(C / groups), (int)(K / groups), (int)RS);
    return hipGetLastError();
}

hipError_t launch_group_dw_extract(const void *full, void *dW, int64_t K, int64_t C, int64_t groups, int64_t RS, hipStream_t s)
{
    const int64_t total = K * (C / groups) * RS;
    const int blocks = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
    hipLaunchKernelGGL(group_dw_extract_kernel, dim3(blocks), dim3(256), 0, s, (const uint32_t *)full, (uint32_t *)dW, (int)K, (int)C,
                       (int)(C / groups), (int)(K / groups), (int)RS);
    return hipGetLastError();
}

hipError_t launch_zero_words(void *p, int64_t n_words, hipStream_t s)
{
    const int fb = (int)((n_words + 255) / 256 < 8192 ? (n_words + 255) / 256 : 8192);
    hipLaunchKernelGGL(zero_words_kernel, dim3(fb < 1 ? 1 : fb), dim3(256), 0, s, (uint32_t *)p, n_words);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Convolution (fast dX kernel: any stride; fast dW kernels: stride 1; the generic kernel serves the rest).
// ------------------------------------------------------------------------------------------------
template <int MODE_G, int MODE_K>
static hipError_t conv_dx_run(const ConvArgs &a, const void *grad, Scale scale, hipStream_t s)
{
    // MODE_G: MODE_BF16 (codes, fp32 weights), MODE_I8 (codes, int8 weights) or MODE_F32 (dense).  MODE_K: the fast kernels'
    // mode, MODE_G itself or MODE_BF16X2 (fp32 weights in two planes).
    if constexpr (MODE_G != MODE_F32) {
        constexpr bool I8 = MODE_G == MODE_I8;
        constexpr int PL = CdxTraits<MODE_K>::PL;
        // The codes as the kernel wants them: planes that start on 4-byte boundaries.  Planes of a size that is not a
        // multiple of 4 (7x7 outputs ...) or a misaligned tensor are copied into padded planes behind the prepared weights.
        const size_t rbw = relayout_bytes(a.K, a.C, a.R, a.S);
        const int64_t PQ = ((a.H + 2 * a.pad - a.R) / a.stride + 1) * ((a.Wd + 2 * a.pad - a.S) / a.stride + 1);
        const int64_t plane = (PQ + 3) / 4 * 4;
        const bool pad_codes = PQ % 4 != 0 || (uintptr_t)grad % 4 != 0;
        const bool codes_ok = !pad_codes || (rbw + (size_t)(a.N * a.K * plane) <= a.scratch_bytes && plane < (1 << 24));
        const int8_t *kernel_codes = pad_codes ? (const int8_t *)a.scratch + rbw : (const int8_t *)grad;
        auto prepare = [&](int taps, int KG, int Cp, const CdxTapMap *map) {
            const int64_t cells = (int64_t)taps * KG * Cp;
            int pb = (int)((cells + 255) / 256 < 4096 ? (cells + 255) / 256 : 4096);
            const int rs = (int)(a.R * a.S);
            // the quantiser's pending statistics sum / bias gradient and the padded copy of the codes ride along in workgroups of their own
            StatsJob job{nullptr, 0, nullptr, nullptr, 0, nullptr, 0.0f, nullptr};
            if (a.pending && (a.pending->n > 0 || a.pending->bias_len > 0)) { job = *a.pending; *a.pending = StatsJob{}; pb += (int)job.workgroups(); }
            CdxPad pad{};
            if (pad_codes) {
                const int64_t dwords = a.N * a.K * (plane / 4), per = dwords < CDX_PAD_TWO ? 256 : 512, wgs = (dwords + per - 1) / per;
                pad = CdxPad{(const int8_t *)grad, (uint32_t *)((char *)a.scratch + rbw), a.N * a.K, (int)PQ, (int)plane, (int)a.K, (int)a.kt(), (int)(wgs < 4096 ? wgs : 4096)};
                pb += pad.workgroups;
            }
            if constexpr (I8) {
                if (map) hipLaunchKernelGGL(conv_dx_weight_prep_i8_kernel<true>, dim3(pb), dim3(256), 0, s, a.W8, (uint4 *)a.scratch, (int)a.K, (int)a.C, taps, KG, Cp, rs, *map, job, pad);
                else     hipLaunchKernelGGL(conv_dx_weight_prep_i8_kernel<false>, dim3(pb), dim3(256), 0, s, a.W8, (uint4 *)a.scratch, (int)a.K, (int)a.C, taps, KG, Cp, rs, CdxTapMap{}, job, pad);
            } else {
                if (map) hipLaunchKernelGGL((conv_dx_weight_prep_kernel<true, PL>), dim3(pb), dim3(256), 0, s, a.W, (uint4 *)a.scratch, (int)a.K, (int)a.C, taps, KG, Cp, rs, *map, job, pad);
                else     hipLaunchKernelGGL((conv_dx_weight_prep_kernel<false, PL>), dim3(pb), dim3(256), 0, s, a.W, (uint4 *)a.scratch, (int)a.K, (int)a.C, taps, KG, Cp, rs, CdxTapMap{}, job, pad);
            }
        };
        if (a.stride != 1 && codes_ok) {
            ConvDxStridedPlan sp = conv_dx_strided_plan(a, I8);
            if (sp.ok && a.plan_only) return hipSuccess;
            if (sp.ok) {
                if (sp.zero_fill && !a.dx_zeroed) {
                    // (one group of a grouped layer never comes here: its dX is not contiguous and the caller has cleared it)
                    const int64_t n = a.N * a.C * a.H * a.Wd;                 // fp32 and int32 zeros are the same bytes
                    const int fb = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
                    hipLaunchKernelGGL(zero_words_kernel, dim3(fb), dim3(256), 0, s, (uint32_t *)a.dX, n);
                }
                if (sp.multi.n > 0) {
                    const int KG = sp.multi.cls[0].KG, Cp = sp.multi.cls[0].Cp;
                    prepare(sp.taps, KG, Cp, &sp.map);
                    for (int i = 0; i < sp.multi.n; ++i) {
                        ConvDxArgs &k = sp.multi.cls[i];
                        k.codes = kernel_codes; k.dX = a.dX; k.scale = scale; k.gate = a.gate;
                        k.code_img = (pad_codes ? a.K : a.kt()) * k.PQ; k.dx_img = a.ct() * k.oPI;
                        k.wp = (const uint4 *)a.scratch + (int64_t)sp.tap_base[i] * KG * PL * Cp;
                    }
                    if (sp.waves) return launch_conv_dx_split(MODE_K, sp.multi, sp.nb, sp.grid, sp.waves, sp.lds_bytes, s);
                    return launch_conv_dx(MODE_K, sp.multi, sp.nb, sp.grid, sp.lds_bytes, s);
                }
                return hipGetLastError();
            }
        }
        ConvDxPlan pl = conv_dx_plan(a, I8);
        if (pl.ok && codes_ok && a.plan_only) return hipSuccess;
        if (pl.ok && codes_ok) {
            ConvDxArgs &k = pl.args;
            k.codes = kernel_codes; k.wp = (const uint4 *)a.scratch; k.dX = a.dX; k.scale = scale; k.gate = a.gate;
            k.code_img = (pad_codes ? a.K : a.kt()) * k.PQ; k.dx_img = a.ct() * k.PI;
            prepare(k.R * k.S, k.KG, k.Cp, nullptr);
            if (pl.waves) return launch_conv_dx_split(MODE_K, k, pl.nb, pl.grid, pl.waves, pl.lds_bytes, s);
            return launch_conv_dx(MODE_K, k, pl.nb, pl.grid, pl.lds_bytes, s);
        }
    }
    if (a.plan_only) { *a.plan_only = 1; return hipSuccess; }         // the generic kernel takes no gate
    ConvGeom g = make_geom(a, ModeTraits<MODE_G>::KCH, k_step<MODE_G>());
    using WT = typename std::conditional<MODE_G == MODE_I8, int8_t, float>::type;      // int8 weights in the full 8-bit mode
    using Acc = typename ModeTraits<MODE_G>::Acc;
    WT *Wt = (WT *)a.scratch;
    const WT *Wsrc = MODE_G == MODE_I8 ? (const WT *)a.W8 : (const WT *)a.W;
    const size_t rb = relayout_bytes(a.K, a.C, a.R, a.S);
    const int64_t total = (int64_t)g.R * g.S * g.Kp * g.C;
    int blocks = (int)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048);
    hipLaunchKernelGGL(conv_weight_relayout_kernel<WT>, dim3(blocks), dim3(256), 0, s, Wsrc, Wt, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int M = g.N * g.H * g.Wd, Kred = g.R * g.S * g.Kp;
    ConvDxGradLoader<MODE_G> al{(const typename GradElem<MODE_G>::T *)grad, g};
    MatrixLoader<MODE_G, false, false> bl{Wt, g.C, g.C, Kred};
    ConvDxOut om{g.Ct, g.H * g.Wd};
    return run_gemm<MODE_G>(al, bl, om, M, g.C, Kred, k_step<MODE_G>(), scale, (Acc *)a.dX,
                            (char *)a.scratch + rb, a.scratch_bytes - rb, s);
}

template <int MODE_G>
static hipError_t conv_dx(const ConvArgs &a, const void *grad, Scale scale, hipStream_t s)
{
    if constexpr (MODE_G == MODE_BF16) {
        if (a.two_planes) return conv_dx_run<MODE_G, MODE_BF16X2>(a, grad, scale, s);
    }
    return conv_dx_run<MODE_G, MODE_G>(a, grad, scale, s);
}

// Which kernel computes a convolution's dW (the same for a launch and for dbp_plan_conv2d_dw), with its plan.
struct ConvDwChoice { int kind; ConvDwPlan p3; ConvDwI8Plan p8; Conv1x1Plan p1; ConvDwtPlan pd; };

template <int MODE>
static ConvDwChoice conv_dw_choose(const ConvArgs &a, const void *grad)
{
    ConvDwChoice c{};
    c.kind = DBP_DW_GENERIC;
    const size_t rb = relayout_bytes(a.K, a.C, a.R, a.S);
    if constexpr (MODE == MODE_I8) {
        c.p8 = conv_dw_i8_plan(a.N, a.C, a.H, a.Wd, a.K, a.R, a.S, a.pad);
        if (c.p8.ok && a.stride == 1 && rb + c.p8.partial_bytes <= a.scratch_bytes && (uintptr_t)a.X % 4 == 0 && (uintptr_t)grad % 4 == 0) {
            c.kind = DBP_DW_3X3_I8;
            return c;
        }
    }
    if constexpr (MODE != MODE_F32) {
        constexpr bool I8 = MODE == MODE_I8;
        ConvDwPlan &pl = c.p3 = conv_dw_plan(a.N, a.C, a.H, a.Wd, a.K, a.R, a.S, a.pad, I8);
        const size_t xal = I8 ? 4 : 16;                              // aligned 4-element loads of both operands
        if (a.stride != 1 || rb + pl.partial_bytes > a.scratch_bytes || (uintptr_t)a.X % xal != 0 || (uintptr_t)grad % 4 != 0) pl.ok = false;
        Conv1x1Plan &p1 = c.p1 = conv1x1_dw_plan(a.N, a.C, a.H, a.Wd, a.K, a.R, a.S, a.pad, a.stride, I8 ? FC2I_KT : FC2_KT);
        if (rb + p1.partial_bytes > a.scratch_bytes) p1.ok = false;
        // The general kernel takes what the two specialised forms do not, and what they are the slower ones for.  Products alone (us), fp32
        // activations (int8 ones lie likewise):
        //   * the 3x3 kernel where its padded rows are more than half (int8: a quarter) full, and small layers; 3x3 kernel / general: 64->64 32x32 52 / 58,
        //     128->128 28x28 60 / 64, 256->256 14x14 64 / 67, narrow rows: 64->64 8x8 N=64 22 / 24, 512->512 4x4 109 / 56,
        //     int8 64->64 4x4 N=128 18 / 29, 512->512 77 / 46;
        //   * the batched 1x1 form by modelled time: 1024->256 14x14 38 / 57, 512->128 28x28 51 / 58, 512->2048 7x7 40 / 55, 64->256 56x56 92 / 39;
        //   * the generic kernel, by modelled time, where up to 16 input channels leave most of the general kernel's blocks of 32 empty: 1->20 5x5
        //     28x28 N=64 34 / 43, 3->64 7x7/2 224x224 N=32 248 / 453, 16->32 3x3/2 32x32 N=128 55 / 34.
        ConvDwtPlan &pd = c.pd;
        if (!(pl.ok && a.Wd * (I8 ? 4 : 2) > pl.args.PW)) {
            pd = conv_dwt_plan(a.N, a.C, a.H, a.Wd, a.K, a.R, a.S, a.pad, a.stride, I8, a.two_planes && !I8 ? 2 : 3);
            // (a group of a grouped layer: images further apart than its own planes say)
            if (pd.ok && (rb + pd.partial_bytes > a.scratch_bytes || pd.args.NI * a.kt() * pd.args.P * pd.args.Q >= ((int64_t)1 << 30) ||
                          pd.args.NI * a.ct() * a.H * a.Wd >= ((int64_t)1 << 29))) pd.ok = false;
            if (pd.ok && pl.ok && pd.us < (I8 ? 17.0f : 12.0f)) pd.ok = false;
            if (pd.ok && p1.ok && p1.us <= 15.0f + pd.us) pd.ok = false;
            // (its own time is about 13 us of ends and 0.8 of the model's)
            if (pd.ok && !pl.ok && !p1.ok && a.C <= 16 && conv_dw_generic_us(a.N, a.C, pd.args.P, pd.args.Q, a.K, a.R * a.S, I8) < 13.0f + 0.8f * pd.us) pd.ok = false;
        }
        c.kind = pd.ok ? DBP_DW_GENERAL : pl.ok ? DBP_DW_3X3 : p1.ok ? DBP_DW_1X1 : DBP_DW_GENERIC;
    }
    return c;
}

template <int MODE>
static hipError_t conv_dw(const ConvArgs &a, const void *grad, Scale scale, hipStream_t s)
{
    using Acc = typename ModeTraits<MODE>::Acc;
    const size_t rb = relayout_bytes(a.K, a.C, a.R, a.S);
    ConvDwChoice c = conv_dw_choose<MODE>(a, grad);
    if (a.plan_only) {
        // the generic kernel takes no gate, and a gate (another kernel may take the product over) is a launch more, 4.5 us: not for the layers
        // that only the general kernel serves
        if (c.kind != DBP_DW_3X3_I8 && !c.p3.ok && !c.p1.ok) *a.plan_only = 1;
        return hipSuccess;
    }
    if constexpr (MODE == MODE_I8) {
        if (c.kind == DBP_DW_3X3_I8) {
            ConvDwI8Args &k = c.p8.args;
            k.codes = (const int8_t *)grad; k.X = (const int8_t *)a.X; k.dW = (int32_t *)a.dW; k.partial = (int32_t *)((char *)a.scratch + rb);
            k.gate = a.gate; k.Ct = (int)a.ct(); k.Kt = (int)a.kt();
            return launch_conv_dw_i8(c.p8, s);
        }
    }
    if constexpr (MODE != MODE_F32) {
        constexpr bool I8 = MODE == MODE_I8;
        if (c.kind == DBP_DW_GENERAL) {
            ConvDwtArgs &k = c.pd.args;
            k.codes = (const int8_t *)grad; k.X = a.X; k.dW = a.dW; k.partial = (char *)a.scratch + rb; k.scale = scale; k.gate = a.gate;
            k.Ct = (int)a.ct(); k.Kt = (int)a.kt();
            if constexpr (I8) return launch_conv_dwt<true, 1>(c.pd, s);
            else return a.two_planes ? launch_conv_dwt<false, 2>(c.pd, s) : launch_conv_dwt<false, 3>(c.pd, s);
        }
        if (c.kind == DBP_DW_3X3) {
            ConvDwArgs &k = c.p3.args;
            k.codes = (const int8_t *)grad; k.X = a.X; k.dW = a.dW; k.partial = (char *)a.scratch + rb; k.scale = scale; k.gate = a.gate;
            k.Ct = (int)a.ct(); k.Kt = (int)a.kt();
            if constexpr (MODE == MODE_BF16) {
                if (a.two_planes)
                    return a.pad == 1 ? launch_conv_dw_fast<MODE_BF16X2, 3, 3, 1, 1>(c.p3, s) : launch_conv_dw_fast<MODE_BF16X2, 3, 3, 0, 1>(c.p3, s);
            }
            return a.pad == 1 ? launch_conv_dw_fast<MODE, 3, 3, 1, 1>(c.p3, s) : launch_conv_dw_fast<MODE, 3, 3, 0, 1>(c.p3, s);
        }
        if (c.kind == DBP_DW_1X1) return launch_conv1x1_dw<I8>(a, c.p1, (const int8_t *)grad, scale, (char *)a.scratch + rb, s);
    }
    ConvGeom g = make_geom(a, ModeTraits<MODE>::KCH, k_step<MODE>());
    const int CRS = g.C * g.R * g.S, Kred = g.N * g.PQp;
    ConvDwGradLoader<MODE> al{(const typename GradElem<MODE>::T *)grad, g};
    ConvDwActLoader<MODE>  bl{(const decltype(ConvDwActLoader<MODE>::base))a.X, g};
    RowMajorOut om{CRS};
    return run_gemm<MODE>(al, bl, om, g.K, CRS, Kred, k_step<MODE>(), scale, (Acc *)a.dW,
                          (char *)a.scratch + rb, a.scratch_bytes - rb, s);
}

static hipError_t conv_products(const ConvArgs &a_in, hipStream_t s)
{
    hipError_t e = hipSuccess;
    const ConvArgs &a = a_in;
    ConvArgs aw = a_in;                                                // what the dW kernels see: their own gate where one is given
    if (a_in.gate_dw.flag) aw.gate = a_in.gate_dw;
    if (a.codes && a.W8) {
        // full 8-bit mode: int8 weights and activations, exact int32 results
        if (a.dX) { e = conv_dx<MODE_I8>(a, a.codes, Scale{1.0f, nullptr}, s); if (e != hipSuccess) return e; }
        if (a.dW) e = conv_dw<MODE_I8>(aw, a.codes, Scale{1.0f, nullptr}, s);
        return e;
    }
    if (a.codes) {
        if (a.dX) { e = conv_dx<MODE_BF16>(a, a.codes, Scale{a.step, a.step_dev}, s); if (e != hipSuccess) return e; }
        if (a.dW) e = a.x_dtype == DBP_F32 ? conv_dw<MODE_BF16>(aw, a.codes, Scale{a.step, a.step_dev}, s) : conv_dw<MODE_I8>(aw, a.codes, Scale{1.0f, nullptr}, s);
        return e;
    }
    if (a.dX) { e = conv_dx<MODE_F32>(a, a.dense, Scale{1.0f, nullptr}, s); if (e != hipSuccess) return e; }
    if (a.dW) e = a.x_dtype == DBP_F32 ? conv_dw<MODE_F32>(aw, a.dense, Scale{1.0f, nullptr}, s) : conv_dw<MODE_I8>(aw, a.dense, Scale{1.0f, nullptr}, s);
    return e;
}

// The quantiser's pending statistics sum and bias gradient go with the first kernel that can take them along (the weight
// preparation of the dX kernels); what nobody took is launched on its own afterwards.
hipError_t launch_conv_mfma(const ConvArgs &a_in, hipStream_t s)
{
    ConvArgs a = a_in;
    StatsJob pending = a_in.stats_job;
    a.pending = &pending;
    hipError_t e = conv_products(a, s);
    if (e == hipSuccess && (pending.n > 0 || pending.bias_len > 0)) e = launch_stats_job(pending, s);
    return e;
}

// ------------------------------------------------------------------------------------------------
// Host-side self-check of the launch plans (no GPU): the planning arithmetic above decides every kernel's indexing, so
// a mistake in it is where an out-of-bounds access would come from.  The checks walk the same functions the launchers
// and the kernels use.  0 = consistent (or the shape takes no planned kernel), otherwise the number of the first
// violated invariant.
// ------------------------------------------------------------------------------------------------
static int check_fc2_pair(int64_t B, int64_t in, int64_t out, bool want_dx, bool want_dw, int kt)
{
    FcPlan pdx, pdw;
    fc2_plans(B, in, out, want_dx, want_dw, pdx, pdw, kt);
    const int64_t items = (want_dx ? pdx.tiles * pdx.n_split : 0) + (want_dw ? pdw.tiles * pdw.n_split : 0);
    if (items > (int64_t)FC2_MAX_ITEMS * 256 || items <= 0) return 0;         // the launcher takes another kernel
    int gx = 0;
    if (want_dx && want_dw) gx = fc2_group_plan(B, in, out, pdx, pdw, kt);
    if (!want_dx) { pdx.n_split = 1; pdx.partial_bytes = 0; }
    if (!want_dw) { pdw.n_split = 1; pdw.partial_bytes = 0; }
    char *scratch = nullptr;
    FcPairArgs pa;
    pa.prob[0] = fc_problem(true, nullptr, out, nullptr, in, (int)B, (int)in, (int)out, Scale{1.0f, nullptr}, nullptr, pdx, scratch);
    pa.prob[1] = fc_problem(false, nullptr, out, nullptr, in, (int)out, (int)in, (int)B, Scale{1.0f, nullptr}, nullptr, pdw, scratch);
    if (!want_dx) pa.prob[0].n_items = 0;
    if (!want_dw) pa.prob[1].n_items = 0;
    pa.gx = gx;
    if ((size_t)(scratch - (char *)nullptr) > linear_scratch_bytes(B, in, out)) return 1;      // partial sums beyond the workspace
    const int total = pa.prob[0].n_items + pa.prob[1].n_items;
    const int G = total < 256 ? total : 256;
    if (gx > 0 && gx >= G) return 2;                                            // the second group would have no workgroup
    std::vector<unsigned char> seen[2];
    seen[0].assign((size_t)pa.prob[0].n_items, 0); seen[1].assign((size_t)pa.prob[1].n_items, 0);
    for (int w = 0; w < G; ++w) {
        const int mine = fc2_items_of_workgroup(pa, G, w);
        if (mine < 0 || mine > FC2_MAX_ITEMS) return 3;
        for (int i = 0; i < mine; ++i) {
            const Fc2Item it = fc2_decode(pa, i, mine, G, w);
            if (it.which < 0 || it.which > 1) return 4;
            const FcProblem &p = pa.prob[it.which];
            if (p.n_items <= 0) return 5;
            const int tiles = p.n_items / p.n_split;
            if (it.tile < 0 || it.tile >= tiles || it.z < 0 || it.z >= p.n_split) return 6;
            if (it.tile_m < 0 || it.tile_m >= p.M || it.tile_n < 0 || it.tile_n >= p.N) return 7;
            if (it.k0 < 0 || it.k0 >= it.k_end || it.k_end > p.K) return 8;
            unsigned char &flag = seen[it.which][(size_t)it.tile * p.n_split + it.z];
            if (flag) return 9;                                                     // an item handed out twice
            flag = 1;
        }
    }
    for (int q = 0; q < 2; ++q)
        for (unsigned char f : seen[q]) if (!f) return 10;                          // an item nobody takes
    return 0;
}

// The direct kernel's plans of a call, made as the launch makes them, with `scratch` bytes for the partial sums.
static int check_fcd(int64_t B, int64_t in, int64_t out, bool want_dx, bool want_dw, bool dx_i8, bool dw_i8, size_t scratch)
{
    size_t left = scratch & ~(size_t)255, used = 0;
    const int room = want_dx && want_dw ? 128 : 256;
    for (int q = 0; q < 2; ++q) {
        const bool kfast = q == 0, i8 = kfast ? dx_i8 : dw_i8;
        const int64_t M = kfast ? B : out, K = kfast ? out : B, kt = i8 ? 32 : 16, tn = fcd_tn(i8), steps = (K + kt - 1) / kt;
        if (!(kfast ? want_dx : want_dw) || !fcd_ok(kfast, M, in, K, out, i8)) continue;
        const FcdPlan pl = fcd_plan(M, in, K, i8, room, left);
        if (pl.us < 0.0f || pl.mf < 1 || pl.mf > (i8 ? 1 : 2) || pl.kw < 1 || pl.kw > FCD_WAVES || (pl.kw & (pl.kw - 1)) || pl.kw > steps) return 12;
        // every tile has its wavefronts, no workgroup is empty, the reduction's parts cover it and none is empty
        if (pl.tiles_m != (M + 32 * pl.mf - 1) / (32 * pl.mf) || pl.tiles != pl.tiles_m * ((in + tn - 1) / tn)) return 13;
        if ((int64_t)pl.groups * FCD_WAVES < (int64_t)pl.tiles * pl.kw || (int64_t)(pl.groups - 1) * FCD_WAVES >= (int64_t)pl.tiles * pl.kw) return 14;
        if ((int64_t)pl.n_split * pl.steps_per_split < steps || (int64_t)(pl.n_split - 1) * pl.steps_per_split >= steps) return 15;
        if (pl.partial_bytes != (pl.n_split > 1 ? (size_t)pl.n_split * M * in * 4 : 0) || used + pl.partial_bytes > scratch) return 16;
        if ((size_t)(FCD_WAVES / 2) * pl.mf * tn * 32 * 4 > (size_t)64 * 1024) return 17;
        // 32-bit lane offsets: a window of rows of the dense operand, the codes
        if (((K < kt ? K : kt) * in + in) * (i8 ? 1 : 4) >= ((int64_t)1 << 32) || (kfast ? M * out : (K < kt ? K : kt) * out + out) >= ((int64_t)1 << 32)) return 18;
        const size_t take = align_up(pl.partial_bytes, 256);
        used += take; left = left > take ? left - take : 0;
    }
    return 0;
}

static int check_conv_plans(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t stride, int64_t pad)
{
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1;
    const size_t total = conv_scratch_bytes(N, C, H, Wd, K, R, S, pad, stride), rb = relayout_bytes(K, C, R, S);
    if (rb > total) return 20;
    ConvArgs a{};
    a.N = N; a.C = C; a.H = H; a.Wd = Wd; a.K = K; a.R = R; a.S = S; a.pad = pad; a.stride = stride;
    for (int i8 = 0; i8 < 2; ++i8) {
        // dX: the stride-1 kernel or the classes of a strided layer
        auto check_dx = [&](const ConvDxArgs &k, int nb, size_t lds, int64_t grid) {
            const int tile_px = k.wpx * 32 * nb;
            if (lds > (size_t)CDX_MAX_LDS || lds < (size_t)2 * CDX_KGC * k.patch_cells * 16) return 21;
            if ((int64_t)k.tiles * tile_px < k.PI || (int64_t)(k.tiles - 1) * tile_px >= k.PI) return 22;      // tiles cover the pixels, none is empty
            if (grid != (int64_t)k.N * k.tiles * k.cgroups || grid <= 0) return 23;
            if (k.wc * k.wpx != 4 || (int64_t)k.cgroups * k.wc * 32 < k.Cp || k.Cp < k.C) return 24;
            if (k.KG % CDX_KGC || (int64_t)k.KG * (i8 ? 16 : 8) < k.K || k.n_chunks * CDX_KGC != k.KG) return 25;
            if ((int64_t)k.prow * k.pw != k.patch_cells || CDX_KGC * (int64_t)k.patch_cells >= 0xFFFF) return 26;
            return 0;
        };
        // ... or, for both, the kernel whose wavefronts divide the reduction
        auto check_split = [&](const ConvDxArgs &k, int nb, int waves, size_t lds, int64_t grid) {
            if ((waves != 4 && waves != 8) || k.pairs < waves || lds > (size_t)CDS_MAX_LDS) return 60;
            if (lds < (size_t)waves * k.wave_cells * 16 || lds < (size_t)waves * nb * 2048 || k.wave_cells != 2 * k.patch_cells + 1 || k.wave_cells >= 0xFFFF) return 61;
            if (k.NI < 1 || (k.NI > 1 && (k.tiles != 1 || k.NI * k.PI > 32 * nb)) || k.NI * k.img_cells != k.patch_cells || k.img_cells != k.prow * k.pw) return 62;
            if ((int64_t)k.tiles * 32 * nb < k.PI || (int64_t)(k.tiles - 1) * 32 * nb >= k.PI) return 63;
            if (grid != (int64_t)((k.N + k.NI - 1) / k.NI) * k.tiles * k.cgroups || k.cgroups * 32 != k.Cp || k.Cp < k.C) return 64;
            const int G = i8 ? 16 : 8;
            if ((int64_t)k.pairs * 2 * G < k.K || (int64_t)(k.pairs - 1) * 2 * G >= k.K || 2 * k.pairs > k.KG) return 65;
            for (int t = 0; t < k.tiles; ++t) {                               // the rows a tile reads: within its patch and its lanes' items
                const int h0 = k.NI > 1 ? 0 : t * 32 * nb / k.Wd, px = k.NI > 1 || (t + 1) * 32 * nb > k.PI ? k.PI : (t + 1) * 32 * nb, h1 = (px - 1) / k.Wd;
                const int lo = h0 + k.pad - (k.R - 1) > 0 ? h0 + k.pad - (k.R - 1) : 0, hi = h1 + k.pad < k.P - 1 ? h1 + k.pad : k.P - 1;
                if (h1 - h0 + k.R > k.prow) return 66;
                if (hi >= lo && 2 * k.NI * (((hi + 1) * k.Q - (lo * k.Q & ~3) + 3) >> 2) > 64 * cds_items(nb)) return 67;
                if (hi >= lo && ((hi + 1) * k.Q + 3) / 4 * 4 > k.PQ) return 68;
            }
            // 32-bit offsets over all images of a tile (the extents are upper bounds of the launch's)
            if ((int64_t)k.NI * k.code_img >= ((int64_t)1 << 31) || (int64_t)k.NI * (k.dx_img + (int64_t)32 * k.oPI) >= ((int64_t)1 << 31)) return 69;
            return 0;
        };
        if (stride == 1) {
            const ConvDxPlan pl = conv_dx_plan(a, i8 != 0);
            if (pl.ok) {
                const int e = pl.waves ? check_split(pl.args, pl.nb, pl.waves, pl.lds_bytes, pl.grid) : check_dx(pl.args, pl.nb, pl.lds_bytes, pl.grid);
                if (e) return e;
            }
        } else {
            const ConvDxStridedPlan sp = conv_dx_strided_plan(a, i8 != 0);
            if (sp.ok) {
                if (sp.multi.n < 0 || sp.multi.n > CDX_MAX_CLASSES || sp.taps > 64) return 27;
                for (int i = 0; i < sp.multi.n; ++i) {
                    const int64_t grid = (int64_t)sp.multi.first[i + 1] - sp.multi.first[i];
                    const int e = sp.waves ? check_split(sp.multi.cls[i], sp.nb, sp.waves, sp.lds_bytes, grid) : check_dx(sp.multi.cls[i], sp.nb, sp.lds_bytes, grid);
                    if (e) return e;
                    if (sp.tap_base[i] + sp.multi.cls[i].R * sp.multi.cls[i].S > sp.taps) return 28;
                }
                if (sp.multi.first[sp.multi.n] != sp.grid) return 29;
                for (int t = 0; t < sp.taps; ++t) if (sp.map.real[t] >= R * S) return 30;
            }
        }
        const size_t padded = (size_t)(N * K * ((P * Q + 3) / 4 * 4));
        if (rb + padded > total) return 31;                                       // the padded copy of the codes
        // dW
        const ConvDwPlan pw = conv_dw_plan(N, C, H, Wd, K, R, S, pad, i8 != 0);
        if (pw.ok && stride == 1) {
            const ConvDwArgs &k = pw.args;
            if (pw.lds_bytes > (size_t)CDW_MAX_LDS || rb + pw.partial_bytes > total) return 32;
            if ((int64_t)k.n_split * k.units_per_split < k.units || (int64_t)(k.n_split - 1) * k.units_per_split >= k.units) return 33;
            if ((int64_t)k.chunks * k.RU < k.H || (int64_t)(k.chunks - 1) * k.RU >= k.H || k.units != N * k.chunks) return 34;
            if ((int64_t)k.tiles_k * 64 * pw.mb < K || (int64_t)k.tiles_c * 64 < C || pw.grid != k.tiles_k * k.tiles_c * k.n_split) return 35;
        }
        if (i8) {
            const ConvDwI8Plan p8 = conv_dw_i8_plan(N, C, H, Wd, K, R, S, pad);
            if (p8.ok && stride == 1) {
                const ConvDwI8Args &k = p8.args;
                if (p8.lds_bytes > (size_t)CDW_MAX_LDS || rb + p8.partial_bytes > total) return 36;
                if ((int64_t)k.n_split * k.units_per_split < k.units || (int64_t)(k.n_split - 1) * k.units_per_split >= k.units) return 37;
                if ((int64_t)k.chunks * k.RU < k.H || k.units != N * k.chunks || k.PW < k.Wd + 1 || k.PW % 16) return 38;
            }
        }
        const Conv1x1Plan p1 = conv1x1_dw_plan(N, C, H, Wd, K, R, S, pad, stride, i8 ? FC2I_KT : FC2_KT);
        if (p1.ok) {
            if (rb + p1.partial_bytes > total) return 39;
            if ((int64_t)p1.n_split * p1.imgs_per_split < N || (int64_t)(p1.n_split - 1) * p1.imgs_per_split >= N) return 40;
            if ((int64_t)p1.spi * p1.kt < H * Wd) return 41;
        }
        for (int planes = i8 ? 3 : 2; planes <= 3; ++planes) {
            const ConvDwtPlan pd = conv_dwt_plan(N, C, H, Wd, K, R, S, pad, stride, i8 != 0, planes);
            if (!pd.ok) continue;
            const ConvDwtArgs &k = pd.args;
            const int RUN = DWT_RUN(i8 != 0), G = pd.G, MF = G == 2 ? 4 : 2, per_chunk = pd.waves / k.chunks;
            const bool one = k.T == 1;
            if (pd.lds_bytes > (size_t)DWT_MAX_LDS || rb + pd.partial_bytes > total) return 42;
            if ((int64_t)k.n_split * k.units_per_split < k.units || (int64_t)(k.n_split - 1) * k.units_per_split >= k.units) return 43;
            // units cover the output, none is empty, and their frames what its taps reach
            if ((int64_t)k.bands * k.PB < P || (int64_t)(k.bands - 1) * k.PB >= P || (int64_t)k.cbands * k.QB < Q || (int64_t)(k.cbands - 1) * k.QB >= Q) return 44;
            if (k.units != (N + k.NI - 1) / k.NI * k.bands * k.cbands || (k.NI > 1 && (k.bands > 1 || k.cbands > 1)) || (k.flat && k.cbands > 1)) return 45;
            if (k.st_lds * k.st_load != stride || (k.st_load > 1 && k.T > 1) || (k.T == 1 && k.frame != k.PB * k.QB)) return 59;   // one tap: no pixel that it does not read
            if (k.frame_w < (k.QB - 1) * k.st_lds + S || (int64_t)k.frame < ((k.PB - 1) * k.st_lds + R) * k.frame_w || (int64_t)k.frame * k.NI > k.chunks * 64) return 46;
            if ((int64_t)k.runs_row * RUN < (k.flat ? (int64_t)k.PB * k.QB : k.QB) || k.runs_img < k.runs_row * (k.flat ? 1 : k.PB) || k.runs_img * k.NI > 2 * k.steps) return 47;
            // wavefronts, channels and taps; staging within a thread's items
            if (k.tg * k.cb * k.kg * k.ps != pd.waves || pd.waves > (one || G == 4 ? 8 : 12) || (k.ps & (k.ps - 1)) || k.chunks > pd.waves) return 48;
            if ((int64_t)k.tiles_k * k.kg * 32 * MF < K || (int64_t)k.tiles_c * k.blocks * 32 < C || k.blocks != k.cb * (one ? G : 1)) return 49;
            if ((int64_t)k.tap_blocks * k.tg * (one ? 1 : G) < k.T || pd.grid != k.tiles_k * k.tiles_c * k.tap_blocks * k.n_split) return 50;
            if (per_chunk * (one ? 6 : 4) < 8 * k.blocks || k.code_step < 1 || k.code_step * 2 * k.steps > 64 * pd.waves ||
                k.code_step * ((one ? 16 : G == 3 ? 8 : 12) / (RUN / 4)) < 32 * MF * k.kg) return 51;
            const int pitch = (i8 ? 32 : 64 * planes) + 8;
            if (k.x_bytes != k.chunks * 64 * pitch * k.blocks || k.buf_bytes != k.x_bytes + 32 * MF * k.kg * (2 * k.steps + 1) * RUN) return 52;
            if (k.last_rows != P - (int64_t)(k.bands - 1) * k.PB || k.last_cols != Q - (int64_t)(k.cbands - 1) * k.QB) return 56;
            if (!i8 && ((k.last_rows < k.PB) != (k.table_row > 0) || (k.last_cols < k.QB) != (k.table_col > 0))) return 57;
            if (k.table_row + k.table_col + 2 * k.steps * RUN > k.tables * 2 * k.steps * RUN || k.table_col % (2 * k.steps * RUN)) return 58;
            if (pd.lds_bytes < (size_t)2 * k.buf_bytes + (size_t)8 * k.steps * RUN * k.tables || pd.lds_bytes < (size_t)(k.ps / 2) * k.tg * k.cb * k.kg * MF * G * 4096) return 53;
            if ((int64_t)(k.NI + 1) * K * P * Q >= ((int64_t)1 << 31) || (int64_t)k.NI * C * H * Wd >= ((int64_t)1 << 29)) return 54;
            if (pd.tch * pd.tap_chunks < k.T || pd.reduce_lds > (size_t)64 * 1024 || pd.reduce_lds < (size_t)pd.zg * 64 * pd.tch * 16) return 55;
        }
    }
    return 0;
}

}  // namespace dbp

extern "C" int dbp_plan_check_linear(int64_t B, int64_t in, int64_t out)
{
    if (B <= 0 || in <= 0 || out <= 0 || B > (1 << 24) || in > (1 << 24) || out > (1 << 24)) return -1;
    for (int kt = dbp::FC2_KT; kt <= dbp::FC2I_KT; kt *= 2)
        for (int m = 1; m < 4; ++m) {
            const int e = dbp::check_fc2_pair(B, in, out, (m & 1) != 0, (m & 2) != 0, kt);
            if (e) return e;
        }
    // the direct kernel: fp32, int8 activations, int8 both; the workspace there is, and next to none
    for (int m = 1; m < 4; ++m)
        for (int i8 = 0; i8 < 3; ++i8)
            for (int small = 0; small < 2; ++small) {
                const int e = dbp::check_fcd(B, in, out, (m & 1) != 0, (m & 2) != 0, i8 == 2, i8 > 0, small ? 1000 : dbp::linear_scratch_bytes(B, in, out));
                if (e) return e;
            }
    // the bias gradient beside a product: 512 columns a workgroup
    dbp::StatsJob job{};
    job.n = 1; job.bias_len = out;
    const int64_t columns = (job.workgroups() - 1) * dbp::StatsJob::kBiasPerGroup;
    if (columns < out || columns - dbp::StatsJob::kBiasPerGroup >= out) return 11;
    return 0;
}

extern "C" int dbp_plan_check_conv2d(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t stride, int64_t pad)
{
    if (N <= 0 || C <= 0 || H <= 0 || Wd <= 0 || K <= 0 || R <= 0 || S <= 0 || stride <= 0 || pad < 0 || H + 2 * pad < R || Wd + 2 * pad < S) return -1;
    if (N > 65535 || C > 65535 || K > 65535 || H > 65535 || Wd > 65535 || R > 255 || S > 255 || pad > 255 || stride > 255) return -1;
    return dbp::check_conv_plans(N, C, H, Wd, K, R, S, stride, pad);
}

extern "C" int dbp_plan_conv2d_dx(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t stride, int64_t pad, int int8_w)
{
    if (dbp_plan_check_conv2d(N, C, H, Wd, K, R, S, stride, pad) != 0) return -1;
    dbp::ConvArgs a{};
    a.N = N; a.C = C; a.H = H; a.Wd = Wd; a.K = K; a.R = R; a.S = S; a.pad = pad; a.stride = stride;
    const dbp::ConvDxPlan pl = dbp::conv_dx_plan(a, int8_w != 0);
    const dbp::ConvDxStridedPlan sp = dbp::conv_dx_strided_plan(a, int8_w != 0);
    if (!pl.ok && !sp.ok) return 0;
    const int nb = pl.ok ? pl.nb : sp.nb, waves = pl.ok ? pl.waves : sp.waves;
    return 16 * waves + nb;
}

extern "C" int dbp_plan_conv2d_dw(int64_t N, int64_t C, int64_t H, int64_t Wd, int64_t K, int64_t R, int64_t S, int64_t stride, int64_t pad,
                                  int int8_x, int dense, int two_planes)
{
    if (dbp_plan_check_conv2d(N, C, H, Wd, K, R, S, stride, pad) != 0) return -1;
    // stand-ins for the tensors: the planners look at alignment only
    char *fake = (char *)(uintptr_t)4096;
    dbp::ConvArgs a{};
    if (dense) a.dense = fake; else a.codes = (const int8_t *)fake;
    a.X = fake; a.dW = fake; a.x_dtype = int8_x ? DBP_I8 : DBP_F32; a.two_planes = two_planes != 0;
    a.N = N; a.C = C; a.H = H; a.Wd = Wd; a.K = K; a.R = R; a.S = S; a.pad = pad; a.stride = stride;
    a.scratch = fake; a.scratch_bytes = dbp::conv_scratch_bytes(N, C, H, Wd, K, R, S, pad, stride);
    if (int8_x) return dbp::conv_dw_choose<dbp::MODE_I8>(a, fake).kind;
    return dense ? dbp::conv_dw_choose<dbp::MODE_F32>(a, fake).kind : dbp::conv_dw_choose<dbp::MODE_BF16>(a, fake).kind;
}

extern "C" int dbp_plan_linear(int64_t B, int64_t in, int64_t out, int int8_x, int int8_w, int want_dx, int want_dw, int two_planes)
{
    if (dbp_plan_check_linear(B, in, out) != 0 || (!want_dx && !want_dw)) return -1;
    char *fake = (char *)(uintptr_t)4096;                            // stand-ins for the tensors
    dbp::LinearArgs a{};
    a.codes = (const int8_t *)fake; a.W8 = int8_w ? (const int8_t *)fake : nullptr; a.x_dtype = int8_x ? DBP_I8 : DBP_F32; a.two_planes = two_planes != 0;
    a.B = B; a.in = in; a.out = out; a.dX = want_dx ? (float *)fake : nullptr; a.dW = want_dw ? fake : nullptr;
    const dbp::FcChoice c = dbp::linear_choose(a);
    auto kind = [](bool want, bool staged, bool direct) { return !want ? 0 : staged ? DBP_FC_STAGED : direct ? DBP_FC_DIRECT : DBP_FC_GENERIC; };
    return kind(want_dx != 0, c.dx_staged, c.dx_direct) | kind(want_dw != 0, c.dw_staged, c.dw_direct) << 4;
}
