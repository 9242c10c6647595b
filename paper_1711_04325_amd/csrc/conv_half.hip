// Launches of the kernels of conv_half.h.
#include "conv_half.h"

namespace rn50 {

void launch_half_prep(const HalfPrep &p, hipStream_t st)
{
    const dim3 gm(p.op[0].blocks + p.op[1].blocks), gs(p.op[0].split_blocks + p.op[1].split_blocks), block(256);
    if (p.in_scale) {
        hipLaunchKernelGGL(half_max_kernel<true>, gm, block, 0, st, p);
        hipLaunchKernelGGL(half_split_kernel<true>, gs, block, 0, st, p);
    } else {
        hipLaunchKernelGGL(half_max_kernel<false>, gm, block, 0, st, p);
        hipLaunchKernelGGL(half_split_kernel<false>, gs, block, 0, st, p);
    }
}

template <int BM, int BN>
static void launch_half(const IgemmWideP &p, int grid, hipStream_t st)
{
    const dim3 g(grid), b(kConvThreads);
    if (p.stat_mean) hipLaunchKernelGGL((igemm_half_kernel<BM, BN, true>), g, b, 0, st, p);
    else hipLaunchKernelGGL((igemm_half_kernel<BM, BN, false>), g, b, 0, st, p);
}
void launch_igemm_half(int bm, int bn, int grid, const IgemmWideP &p, hipStream_t st)
{
    if (bm == 128) launch_half<128, 64>(p, grid, st);
    else if (bn == 128) launch_half<64, 128>(p, grid, st);
    else launch_half<64, 64>(p, grid, st);
}

}  // namespace rn50
