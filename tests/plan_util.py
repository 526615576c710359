"""The kernels that the library would choose (host only): what a test that aims at one of them asserts."""
import ctypes as C

import paper_2004_04729_amd as dbp

GENERIC_FC, DIRECT, STAGED = 1, 2, 3                              # DBP_FC_*
GENERIC, THREE, THREE_I8, ONE, GENERAL = range(5)                 # DBP_DW_*


def fc_kernels(B, in_, out, i8=0, q8=0, dx=1, dw=1, two=0):
    """Kernels of (dX, dW); None for a product that is not asked for."""
    f = dbp.lib().dbp_plan_linear
    f.argtypes, f.restype = [C.c_int64] * 3 + [C.c_int] * 5, C.c_int
    r = f(B, in_, out, i8 or q8, q8, dx, dw, two)
    return (r & 15) or None, (r >> 4) or None


def conv_dw_kernel(N, C_, H, Wd, K, R, S, stride, pad, i8=0, dense=0, two=0):
    f = dbp.lib().dbp_plan_conv2d_dw
    f.argtypes, f.restype = [C.c_int64] * 9 + [C.c_int] * 3, C.c_int
    return f(N, C_, H, Wd, K, R, S, stride, pad, i8, dense, two)


def conv_dx_kernel(N, C_, H, Wd, K, R, S, stride, pad, q8=0):
    """0: generic, else (wavefronts that divide the reduction, pixel blocks); wavefronts 0: the kernel that divides channels and pixels."""
    f = dbp.lib().dbp_plan_conv2d_dx
    f.argtypes, f.restype = [C.c_int64] * 9 + [C.c_int], C.c_int
    r = f(N, C_, H, Wd, K, R, S, stride, pad, q8)
    return divmod(r, 16) if r > 0 else r
