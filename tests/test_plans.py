"""Host-side walk of the launch plans (no GPU): for a grid of layer shapes, the planning code of the fast kernels must hand
out every work item exactly once, keep every tile / split / class index in range and every partial-sum buffer inside
the workspace size the library reports.  This is the arithmetic a GPU fault would come from."""
import ctypes as C
import itertools
import time

import pytest

import paper_2004_04729_amd as dbp
from plan_util import DIRECT, GENERAL, GENERIC, GENERIC_FC, ONE, STAGED, THREE, conv_dw_kernel as _dw, conv_dx_kernel as _dx, fc_kernels as _fc


def _lib():
    L = dbp.lib()
    L.dbp_plan_check_linear.argtypes = [C.c_int64] * 3
    L.dbp_plan_check_conv2d.argtypes = [C.c_int64] * 9
    return L


FC_DIMS = [1, 2, 3, 4, 31, 32, 33, 64, 100, 127, 128, 129, 255, 256, 257, 300, 511, 512, 513, 784, 1000, 1024, 1030, 2048, 4096, 4100, 8192]


def test_fc_plans_cover_every_item_once_and_stay_in_bounds():
    L = _lib()
    bad = []
    for B, in_, out in itertools.product(FC_DIMS, FC_DIMS, FC_DIMS):
        e = L.dbp_plan_check_linear(B, in_, out)
        if e:
            bad.append((B, in_, out, e))
    assert not bad, bad[:10]
    # the configurations and a few very large layers
    for B, in_, out in [(64, 784, 300), (256, 1024, 4096), (256, 4096, 4096), (256, 4096, 1000), (256, 8192, 8192), (300, 4096, 4000),
                        (2048, 2048, 2048), (256, 4096, 16384), (65536, 65536, 8), (8, 65536, 65536), (4096, 16384, 16384)]:
        assert L.dbp_plan_check_linear(B, in_, out) == 0, (B, in_, out)
    assert L.dbp_plan_check_linear(0, 4, 4) == -1


def test_fc_kernels_are_the_faster_ones():
    """The choice between the direct and the staged kernel on layers where both were measured (us; dX direct and dW staged: mixed)."""
    D, S = DIRECT, STAGED
    for case, want in [((128, 8192, 8192), (S, S)),          # staged 160, direct 281
                       ((96, 8192, 8192), (D, S)),           # mixed 153, staged 162, direct 261
                       ((32, 8192, 8192), (D, S)),           # mixed 105, staged 141, direct 146
                       ((128, 4096, 4096), (S, S)),          # 49, direct 56
                       ((64, 4096, 4096), (D, D)),           # 43, mixed 44, staged 56
                       ((4096, 8192, 100), (S, S)), ((4096, 8192, 64), (S, D)), ((2048, 4096, 16), (D, D)),      # 82 / 116, 66 / 81
                       ((256, 4096, 4096), (S, S)), ((256, 1024, 4096), (S, S)), ((256, 1024, 1024), (D, D)), ((64, 784, 300), (D, D))]:
        assert _fc(*case) == want, case
    for case, want in [((128, 8192, 8192), (S, S)), ((96, 4096, 16384), (D, S)), ((128, 8192, 4096), (D, D)), ((128, 4096, 4096), (D, D)), ((256, 4096, 4096), (S, S))]:
        assert _fc(*case, q8=1) == want, case
    # a product alone
    assert _fc(64, 2048, 2048, dx=0) == (None, S) and _fc(32, 1024, 1024, dx=0) == (None, D)                            # 11 / 13, 9 / 8
    assert _fc(512, 8192, 64, dw=0) == (S, None) and _fc(64, 4096, 4096, dw=0) == (D, None)                              # 11 / 13, 37 / 25
    assert _fc(4, 1, 4) == (GENERIC_FC, GENERIC_FC)
    # two planes: the staged kernel wherever both products fill a tile
    assert _fc(256, 300, 300, two=1) == (S, S) and _fc(64, 300, 300, two=1) == (D, D)


CONV = [  # N, C, H, Wd, K, R, S, stride, pad
    (128, 64, 32, 32, 64, 3, 3, 1, 1), (64, 256, 14, 14, 256, 3, 3, 1, 1), (64, 1024, 14, 14, 256, 1, 1, 1, 0), (32, 256, 56, 56, 256, 3, 3, 1, 1),
    (64, 128, 28, 28, 256, 3, 3, 2, 1), (64, 256, 14, 14, 512, 3, 3, 2, 1), (64, 3, 224, 224, 64, 7, 7, 2, 3), (32, 64, 15, 15, 64, 3, 3, 1, 1),
    (16, 512, 7, 7, 512, 3, 3, 1, 1), (8, 96, 27, 27, 256, 5, 5, 1, 2), (1, 1, 1, 1, 1, 1, 1, 1, 0), (2, 5, 9, 7, 6, 3, 3, 1, 1),
    (64, 132, 24, 20, 264, 1, 1, 2, 0), (1, 8, 17, 17, 8, 3, 3, 4, 1), (2, 16, 9, 224, 8, 3, 3, 1, 1), (1, 16, 20, 228, 16, 3, 3, 1, 1),
]


def test_conv_plans_stay_in_bounds():
    L = _lib()
    for case in CONV:
        assert L.dbp_plan_check_conv2d(*case) == 0, case
    bad = []
    for N, C_, H, K, (R, st, pad) in itertools.product([1, 3, 32, 70], [1, 3, 16, 33, 64, 130, 256], [1, 5, 7, 8, 14, 15, 28, 31, 56],
                                                        [1, 8, 20, 64, 130, 260], [(1, 1, 0), (3, 1, 1), (3, 1, 0), (3, 2, 1), (5, 1, 2), (7, 2, 3), (2, 2, 0), (3, 3, 0)]):
        for Wd in {H, H + 3, 4 * ((H + 3) // 4)}:
            if H + 2 * pad < R or Wd + 2 * pad < R:
                continue
            e = L.dbp_plan_check_conv2d(N, C_, H, Wd, K, R, R, st, pad)
            if e:
                bad.append((N, C_, H, Wd, K, R, st, pad, e))
    assert not bad, bad[:10]
    assert L.dbp_plan_check_conv2d(1, 1, 2, 2, 1, 5, 5, 1, 0) == -1


def test_conv_dw_of_dense_int8_runs_where_that_of_codes_does():
    # an int8 gradient is an int8 gradient: strided layers, odd planes, odd kernels and 1x1 layers leave the generic kernel
    for case in CONV:
        assert _dw(*case, i8=1, dense=1) == _dw(*case, i8=1), case
    for case in [(64, 128, 28, 28, 256, 3, 3, 2, 1), (64, 512, 7, 7, 512, 3, 3, 1, 1), (32, 96, 27, 27, 256, 5, 5, 1, 2), (64, 512, 14, 14, 1024, 1, 1, 2, 0)]:
        assert _dw(*case, i8=1, dense=1) == GENERAL, case
        assert _dw(*case, dense=1) == GENERIC, case                    # fp32 gradients have no other
    assert _dw(1, 1, 2, 2, 1, 5, 5, 1, 0) == -1


def test_conv_dw_kernels_are_the_faster_ones():
    """The choice between the kernels for dW on layers where each was measured (the product alone, the next best kernel's time
    in parentheses, us)."""
    for want, cases in {
        GENERIC: [(64, 1, 28, 28, 20, 5, 5, 1, 0),          # 34 (general 43): one input channel in a block of 32
                  (32, 3, 224, 224, 64, 7, 7, 2, 3),        # 248 (453)
                  (128, 1, 64, 64, 32, 5, 5, 2, 2),         # 59 (102)
                  (1, 1, 12, 12, 64, 5, 5, 2, 0)],          # 10 (24)
        GENERAL: [(64, 128, 28, 28, 256, 3, 3, 2, 1), (16, 64, 56, 56, 64, 5, 5, 1, 2), (32, 64, 56, 56, 256, 1, 1, 1, 0),
                  (128, 16, 32, 32, 32, 3, 3, 2, 1), (128, 512, 4, 4, 512, 3, 3, 1, 1), (64, 512, 14, 14, 1024, 1, 1, 2, 0)],
        ONE: [(64, 1024, 14, 14, 256, 1, 1, 1, 0), (64, 128, 28, 28, 512, 1, 1, 1, 0), (64, 512, 7, 7, 2048, 1, 1, 1, 0),      # 43 (52), 40 (55)
              (61, 104, 8, 8, 232, 1, 1, 1, 0), (10, 128, 16, 16, 992, 1, 1, 1, 0)],                                   # 17 (22), 19 (27)
        THREE: [(128, 64, 32, 32, 64, 3, 3, 1, 1), (64, 256, 14, 14, 256, 3, 3, 1, 1),
                (20, 88, 8, 8, 32, 3, 3, 1, 1), (64, 64, 8, 8, 64, 3, 3, 1, 1)],                                       # 17 (20), 21 (24): small layers
    }.items():
        for case in cases:
            assert _dw(*case) == want, (case, _dw(*case), want)
    # int8 activations: 28 (40), 24 (40), 15 (20), 18 (20); 30 (41) the other way round
    for case in [(64, 1024, 14, 14, 256, 1, 1, 1, 0), (64, 128, 28, 28, 512, 1, 1, 1, 0), (16, 216, 40, 40, 72, 1, 1, 1, 0), (28, 20, 20, 20, 146, 1, 1, 1, 0)]:
        assert _dw(*case, i8=1) == ONE, case
    assert _dw(1, 1, 12, 12, 64, 5, 5, 2, 0, i8=1) == GENERIC
    assert _dw(128, 64, 4, 4, 64, 3, 3, 1, 1, i8=1) == THREE and _dw(128, 512, 4, 4, 512, 3, 3, 1, 1, i8=1) == GENERAL      # 18 (29); 46 (77)


def test_conv_planning_time_does_not_grow_with_the_plane():
    """Planning is host time of every call.  A 2048x2048 plane has 1000 times the tiles of a 64x64 one, and no tile of it fits: a
    planner that walks them all takes over 100 times as long, one that stops at the first no longer than for the small plane."""
    f = dbp.lib().dbp_plan_auto_conv2d
    f.argtypes, f.restype = [C.c_int64] * 9 + [C.c_int] * 4 + [C.POINTER(C.c_uint64)] * 2, C.c_int
    a, b = C.c_uint64(), C.c_uint64()

    def microseconds(*case):
        best = 1e9
        for _ in range(9):
            t = time.perf_counter()
            for _ in range(10):
                f(*case, 0, 1, 0, 0, C.byref(a), C.byref(b))
            best = min(best, (time.perf_counter() - t) * 1e5)
        return best

    for K in (16, 256):
        assert microseconds(1, 16, 2048, 2048, K, 3, 3, 1, 1) < 10 * microseconds(1, 16, 64, 64, K, 3, 3, 1, 1)
    assert microseconds(1, 64, 2048, 2048, 256, 3, 3, 2, 1) < 10 * microseconds(1, 64, 64, 64, 256, 3, 3, 2, 1)


def test_conv_dx_kernels_are_the_faster_ones():
    """The choice between the two dX kernels, and of tile and wavefronts, on layers where the forms were measured (us)."""
    for case, want in [((3, 88, 147, 147, 432, 2, 2, 2, 1), (0, 2)),       # int8 weights, strided: 44, the other kernel's 7 blocks x 4 wavefronts 61
                       ((8, 49, 197, 197, 499, 2, 2, 2, 1), (0, 2)),       # 191, 4x4 248
                       ((96, 24, 145, 7, 188, 3, 3, 3, 2), (0, 2)),       # 30, 7x4 38
                       ((51, 24, 90, 90, 336, 2, 2, 2, 1), (0, 2)),       # 101, 7x4 125
                       ((70, 427, 20, 7, 475, 3, 3, 2, 1), (4, 4)),       # 50, 7x8 64; 55
                       ((3, 16, 23, 23, 864, 3, 3, 2, 1), (8, 2)),        # 22; 47
                       ((3, 512, 18, 18, 792, 3, 3, 2, 1), (8, 4))]:      # 26; 52
        assert _dx(*case, q8=1) == want, case
    for case, want in [((64, 256, 14, 14, 256, 3, 3, 1, 1), (4, 7)), ((64, 512, 7, 7, 512, 3, 3, 1, 1), (8, 7)),         # 48; 66.  53; 82
                       ((119, 16, 8, 8, 537, 3, 3, 1, 1), (8, 2)), ((83, 40, 8, 8, 840, 3, 3, 2, 1), (8, 2)),           # 22; 70.  27; 81
                       ((128, 64, 32, 32, 64, 3, 3, 1, 1), (0, 4)), ((64, 1024, 14, 14, 256, 1, 1, 1, 0), (0, 7))]:     # 39; 50.  34
        assert _dx(*case) == want, case


def test_conv_dx_tile_of_few_images_where_offsets_would_pass_31_bits():
    """One pixel an image under a padding of 100: 20000 planes of 201x201 codes, 0.8e9 codes an image.  Three images fit a lane's items and
    would pass 2^31 (dbp_plan_check_conv2d answers 69 for such a tile); two do not."""
    case = (600, 8, 1, 1, 20000, 1, 1, 1, 100)
    assert _lib().dbp_plan_check_conv2d(*case) == 0 and _dx(*case) == (8, 2)


def test_conv_dx_of_layers_that_fit_no_tile_is_generic():
    """Stride 4 has no class plan; 3x3 rows of 700 codes exceed a workgroup's patch in every form of both kernels."""
    for q8 in (0, 1):
        for case in [(2, 8, 19, 19, 64, 3, 3, 4, 1), (2, 64, 700, 700, 128, 3, 3, 1, 1), (2, 64, 1400, 1400, 128, 3, 3, 2, 1)]:
            assert _dx(*case, q8=q8) == 0, case


def test_conv_gather_plans_stay_in_bounds():
    # the gather kernels that scan the code planes: bands, tiles, LDS sizes, the reciprocals that replace divisions
    L = dbp.lib()
    L.dbp_plan_check_conv2d_gather.argtypes = [C.c_int64] * 9 + [C.c_int, C.c_size_t]
    big = 1 << 30
    for case in CONV:
        for i8 in (0, 1):
            for scratch in (0, 1 << 20, big):
                assert L.dbp_plan_check_conv2d_gather(*case, i8, scratch) == 0, (case, i8, scratch)
    bad = []
    for N, C_, H, K, (R, st, pad) in itertools.product([1, 3, 32, 70], [1, 16, 33, 64, 130, 256], [1, 2, 4, 6, 8, 14, 16, 28, 30, 56, 112],
                                                        [1, 8, 33, 64, 130, 260], [(1, 1, 0), (3, 1, 1), (3, 1, 0), (3, 2, 1), (3, 1, 2), (1, 2, 0)]):
        for Wd in {H, H + 2, 4 * ((H + 3) // 4), 200, 252}:
            if H + 2 * pad < R or Wd + 2 * pad < R:
                continue
            for i8 in (0, 1):
                e = L.dbp_plan_check_conv2d_gather(N, C_, H, Wd, K, R, R, st, pad, i8, big)
                if e:
                    bad.append((N, C_, H, Wd, K, R, st, pad, i8, e))
    assert not bad, bad[:10]
    assert L.dbp_plan_check_conv2d_gather(1, 1, 2, 2, 1, 5, 5, 1, 0, 0, 0) == -1


def test_conv_auto_plan_arms_what_the_measurements_say():
    """The host's cost models behind DBP_PATH_AUTO on the layer shapes they were calibrated on (measured on MI355X: where the
    plane-scanning gather kernel for dW beats the matrix cores below 2-4 % nonzeros it is armed, with a threshold in that
    range; where it never does, or the gate's empty launches would cost more than it can win, nothing is armed)."""
    L = _lib()
    L.dbp_plan_auto_conv2d.argtypes = [C.c_int64] * 9 + [C.c_int] * 4 + [C.POINTER(C.c_uint64)] * 2
    L.dbp_plan_auto_conv2d.restype = C.c_int

    def plan(N, C_, H, K, R, pad, i8=0, dx=1, dw=1, two=0, stride=1):
        g, d = C.c_uint64(7), C.c_uint64(7)
        kind = L.dbp_plan_auto_conv2d(N, C_, H, H, K, R, R, stride, pad, i8, dx, dw, two, C.byref(g), C.byref(d))
        codes = N * K * ((H + 2 * pad - R) // stride + 1) ** 2
        return kind, g.value / codes, d.value / codes

    # dW alone on the gather kernel: armed, switching between 1.5 % and 5 % nonzeros (measured crossovers: 3-4 %)
    for shape in [(64, 256, 14, 256), (64, 512, 14, 512), (32, 256, 28, 256), (16, 128, 56, 128), (256, 128, 16, 128)]:
        kind, g, d = plan(*shape, 3, 1)
        assert kind == 2 and g == 0 and 0.015 < d < 0.05, (shape, kind, g, d)
        assert plan(*shape, 3, 1, dx=0)[0] == 2                         # also for a call that asks for dW alone
        assert plan(*shape, 3, 1, dw=0)[0] in (0, 1)                    # and never for one that asks for dX alone
    # too little to win (64-channel layers, config 3's shape among them; 1x1 layers): no gate, or the whole-family one
    for shape, r, pad in [((128, 64, 32, 64), 3, 1), ((32, 64, 56, 64), 3, 1), ((64, 1024, 14, 256), 1, 0), ((32, 512, 28, 128), 1, 0)]:
        kind, g, d = plan(*shape, r, pad)
        assert kind in (0, 1) and d == 0, (shape, kind, d)
    # int8 activations keep dW on the int8 matrix cores: config 5 no gate at all, the 14x14 layer the whole-family gate beyond 99.5 % zeros
    assert plan(32, 256, 56, 256, 3, 1, i8=1)[0] == 0
    kind, g, d = plan(64, 256, 14, 256, 3, 1, i8=1)
    assert kind == 1 and d == 0 and 0 < g < 0.005, (kind, g, d)
    # shapes the kernels decline (stride 2; 5x5) and invalid ones
    assert plan(64, 256, 28, 256, 3, 1, stride=2)[0] in (0, 1) and plan(16, 64, 28, 64, 5, 2)[0] in (0, 1)
    assert L.dbp_plan_auto_conv2d(1, 1, 2, 2, 1, 5, 5, 1, 0, 0, 1, 1, 0, None, None) == -1
    assert L.dbp_plan_auto_conv2d(4, 8, 8, 8, 8, 3, 3, 1, 1, 0, 0, 0, 0, None, None) == -1


def test_conv_auto_plan_counts_the_walk_over_an_images_entries():
    """Few images: dX's gather workgroups walk an image's entries one after the other (0.21 us each).  Layers timed on both sides (us): the
    threshold lies below the density at which the gather family was the slower one."""
    f = dbp.lib().dbp_plan_auto_conv2d
    f.argtypes, f.restype = [C.c_int64] * 9 + [C.c_int] * 4 + [C.POINTER(C.c_uint64)] * 2, C.c_int
    for case, dw, nonzero in [((10, 80, 6, 153, 936, 3, 3, 1, 1), 0, 0.0008),          # gather 257, matrix cores 112
                              ((5, 248, 26, 26, 624, 3, 3, 1, 1), 1, 0.0009),          # 171, 112
                              ((2, 561, 9, 60, 744, 3, 3, 1, 1), 1, 0.0009)]:          # 186, 143
        g, d = C.c_uint64(), C.c_uint64()
        N, _, H, Wd, K = case[:5]
        assert f(*case, 0, 1, dw, 0, C.byref(g), C.byref(d)) == 1 and 0 < g.value < nonzero * N * K * H * Wd, case


def test_fc_auto_plan_arms_the_wide_layer_only():
    """Fully connected layers: the gather family's fixed cost (streaming the dense operand, writing dW) is what the matrix
    cores pay too, so the gate is armed only where a layer is wide enough for the nonzero-proportional part to matter:
    256x4096x16384 (measured: gather wins from ~98.5 % zeros), not the 4096-wide layers of the MLP or 2048^3."""
    L = _lib()
    L.dbp_plan_auto_linear.argtypes = [C.c_int64] * 3 + [C.c_int] * 4 + [C.POINTER(C.c_uint64)]
    L.dbp_plan_auto_linear.restype = C.c_int
    g = C.c_uint64(7)
    assert L.dbp_plan_auto_linear(256, 4096, 16384, 0, 1, 1, 0, C.byref(g)) == 1
    assert 0.005 < g.value / (256 * 16384) < 0.03, g.value
    for B, in_, out in [(256, 4096, 4096), (256, 784, 4096), (256, 4096, 1000), (2048, 2048, 2048), (64, 784, 300)]:
        assert L.dbp_plan_auto_linear(B, in_, out, 0, 1, 1, 0, C.byref(g)) == 0 and g.value == 0, (B, in_, out)
    assert L.dbp_plan_auto_linear(0, 4, 4, 0, 1, 1, 0, None) == -1
