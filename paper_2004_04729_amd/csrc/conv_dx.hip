// Launches of conv_dx_kernel and conv_dx_multi_kernel; plans: products.hip, the kernel that divides the reduction: conv_dx_split.hip.  A code object of its
// own: among the dW kernels of products.hip its loops cost calls of those up to 2 % (512->512 7x7 N=64, the call: 126.5 us and 129.4).
#include <hip/hip_runtime.h>
#include "conv_dx_kernel.h"

namespace dbp {

template <int MODE>
static void launch_mode(const ConvDxArgs &args, int nb, int grid, size_t lds, hipStream_t s)
{
    const int taps = args.R * args.S;
    auto launch = [&](auto n, auto form) {
        hipLaunchKernelGGL((conv_dx_kernel<decltype(n)::value, MODE, decltype(form)::value>), dim3(grid), dim3(256), lds, s, args);
    };
    auto blocks = [&](auto form) {
        if (nb == 7)      launch(std::integral_constant<int, 7>{}, form);
        else if (nb == 4) launch(std::integral_constant<int, 4>{}, form);
        else              launch(std::integral_constant<int, 2>{}, form);
    };
    if (taps == 1)          blocks(std::integral_constant<int, 1>{});
    else if (taps % 3 == 0) blocks(std::integral_constant<int, 3>{});
    else                    blocks(std::integral_constant<int, 0>{});
}

template <int MODE>
static void launch_mode(const ConvDxMulti &args, int nb, int grid, size_t lds, hipStream_t s)
{
    auto launch = [&](auto n, auto form) {
        hipLaunchKernelGGL((conv_dx_multi_kernel<decltype(n)::value, MODE, decltype(form)::value>), dim3(grid), dim3(256), lds, s, args);
    };
    auto blocks = [&](auto form) {
        if (nb == 7)      launch(std::integral_constant<int, 7>{}, form);
        else if (nb == 4) launch(std::integral_constant<int, 4>{}, form);
        else              launch(std::integral_constant<int, 2>{}, form);
    };
    // (a 1x1 kernel: the one class that has a tap)
    if (MODE != MODE_I8 && args.n == 1 && args.cls[0].R * args.cls[0].S == 1) blocks(std::integral_constant<int, MODE == MODE_I8 ? 0 : 1>{});
    else                                                                      blocks(std::integral_constant<int, 0>{});
}

hipError_t launch_conv_dx(int mode, const ConvDxArgs &args, int nb, int grid, size_t lds, hipStream_t s)
{
    if (mode == MODE_I8)          launch_mode<MODE_I8>(args, nb, grid, lds, s);
    else if (mode == MODE_BF16X2) launch_mode<MODE_BF16X2>(args, nb, grid, lds, s);
    else                          launch_mode<MODE_BF16>(args, nb, grid, lds, s);
    return hipGetLastError();
}

hipError_t launch_conv_dx(int mode, const ConvDxMulti &args, int nb, int grid, size_t lds, hipStream_t s)
{
    if (mode == MODE_I8)          launch_mode<MODE_I8>(args, nb, grid, lds, s);
    else if (mode == MODE_BF16X2) launch_mode<MODE_BF16X2>(args, nb, grid, lds, s);
    else                          launch_mode<MODE_BF16>(args, nb, grid, lds, s);
    return hipGetLastError();
}

}  // namespace dbp
