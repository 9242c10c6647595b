// Launches of the first layer's kernels (conv_stem.h).
#include "conv_stem.h"

#include <algorithm>

namespace rn50 {

template <int PREC>
static void launch_fwd(bool stats, const StemMP &p, hipStream_t st)
{
    const dim3 grid(std::min(p.ntiles, (PREC == 2 ? 2 : 3) * 256)), block(kConvThreads);  // 256 CUs
    if (stats) hipLaunchKernelGGL((stem_mm_fwd_kernel<PREC, true>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((stem_mm_fwd_kernel<PREC, false>), grid, block, 0, st, p);
}
void launch_stem_fwd(int prec, bool stats, const StemMP &p, hipStream_t st)
{
    if (prec == 2) launch_fwd<2>(stats, p, st);
    else launch_fwd<1>(stats, p, st);
}
void launch_stem_wgrad(int prec, int grid, const StemWP &p, hipStream_t st)
{
    if (prec == 2) hipLaunchKernelGGL((stem_mm_wgrad_kernel<2>), dim3(grid), dim3(kConvThreads), 0, st, p);
    else hipLaunchKernelGGL((stem_mm_wgrad_kernel<1>), dim3(grid), dim3(kConvThreads), 0, st, p);
}

}  // namespace rn50
