// Launches of the kernel of conv_small.h.
#include "conv_small.h"

namespace rn50 {

template <int TM, int TN>
static void launch_small(const IgemmWideP &p, int grid, hipStream_t st)
{
    const dim3 g(grid), b(64 * kSmallWaves);
    if (p.flip_taps) hipLaunchKernelGGL((igemm_small_kernel<TM, TN, true, false, false>), g, b, 0, st, p);
    else if (p.in_scale && p.stat_mean) hipLaunchKernelGGL((igemm_small_kernel<TM, TN, false, true, true>), g, b, 0, st, p);
    else if (p.in_scale) hipLaunchKernelGGL((igemm_small_kernel<TM, TN, false, true, false>), g, b, 0, st, p);
    else if (p.stat_mean) hipLaunchKernelGGL((igemm_small_kernel<TM, TN, false, false, true>), g, b, 0, st, p);
    else hipLaunchKernelGGL((igemm_small_kernel<TM, TN, false, false, false>), g, b, 0, st, p);
}
// bm, bn: rows and columns of a workgroup, 16 or 32 each
void launch_igemm_small(int bm, int bn, int grid, const IgemmWideP &p, hipStream_t st)
{
    if (bm == 32 && bn == 32) launch_small<2, 2>(p, grid, st);
    else if (bm == 32) launch_small<2, 1>(p, grid, st);
    else if (bn == 32) launch_small<1, 2>(p, grid, st);
    else launch_small<1, 1>(p, grid, st);
}

}  // namespace rn50
