// Launches of conv_dx_split_kernel (its plans: products.hip).  A source file and so a code object of its own: emitted among the kernels of products.hip,
// its 26 instantiations lay between those that one call runs in turn, and calls that never use them took longer (1x1 2048->512 7x7
// N=32, the call: 65.4 us without the kernel, 66.6 among the others, 65.2 here; 1x1 1024->256 14x14 N=64: 86.5, 86.8, 86.65).
#include <hip/hip_runtime.h>
#include "conv_dx_split_kernel.h"

namespace dbp {

template <class Args>
static hipError_t launch_as(void (*kernel)(Args), bool &raised, const Args &args, int grid, int waves, size_t lds, hipStream_t s)
{
    if (!raised) {                                                   // more than 64 KiB of dynamic LDS: allowed per kernel, once
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, CDS_MAX_LDS);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * waves), lds, s, args);
    return hipGetLastError();
}

template <int NB, int MODE>
static hipError_t launch_nb(const ConvDxArgs &args, int grid, int waves, size_t lds, hipStream_t s)
{
    static bool raised[2] = {false, false};
    // Seven blocks and sixteen raw dwords an item do not fit the registers: unrolled not at all, and rolled one is spilled, outside the loops.
    if constexpr (NB < 7 || MODE != MODE_I8) {
        if (args.R == 3 && args.S == 3) return launch_as(&conv_dx_split_kernel<NB, MODE, true>, raised[1], args, grid, waves, lds, s);
    }
    return launch_as(&conv_dx_split_kernel<NB, MODE, false>, raised[0], args, grid, waves, lds, s);
}

template <int NB, int MODE>
static hipError_t launch_nb(const ConvDxMulti &args, int grid, int waves, size_t lds, hipStream_t s)
{
    // (int8 with seven blocks: spilled registers, too, and of 566 strided layers the fastest form for so few that leaving it out of the choice made
    // the choice better: planned never)
    if constexpr (NB == 7 && MODE == MODE_I8) return hipErrorInvalidValue;
    static bool raised = false;
    return launch_as(&conv_dx_split_multi_kernel<NB, MODE>, raised, args, grid, waves, lds, s);
}

template <int MODE, class Args>
static hipError_t launch_mode(const Args &args, int nb, int grid, int waves, size_t lds, hipStream_t s)
{
    return nb == 7 ? launch_nb<7, MODE>(args, grid, waves, lds, s) : nb == 4 ? launch_nb<4, MODE>(args, grid, waves, lds, s) : launch_nb<2, MODE>(args, grid, waves, lds, s);
}

template <class Args>
static hipError_t launch(int mode, const Args &args, int nb, int grid, int waves, size_t lds, hipStream_t s)
{
    return mode == MODE_I8 ? launch_mode<MODE_I8>(args, nb, grid, waves, lds, s) :
           mode == MODE_BF16X2 ? launch_mode<MODE_BF16X2>(args, nb, grid, waves, lds, s) : launch_mode<MODE_BF16>(args, nb, grid, waves, lds, s);
}

hipError_t launch_conv_dx_split(int mode, const ConvDxArgs &args, int nb, int grid, int waves, size_t lds, hipStream_t s)
{
    return launch(mode, args, nb, grid, waves, lds, s);
}

hipError_t launch_conv_dx_split(int mode, const ConvDxMulti &args, int nb, int grid, int waves, size_t lds, hipStream_t s)
{
    return launch(mode, args, nb, grid, waves, lds, s);
}

}  // namespace dbp
