// Launches of the kernels of conv_terms.h.
#include "conv_terms.h"

namespace rn50 {

void launch_terms_prep(const TermsPrep &p, hipStream_t st)
{
    const dim3 grid(p.blocks[0] + p.blocks[1]), block(256);
    if (p.in_scale) hipLaunchKernelGGL(terms_prep_kernel<true>, grid, block, 0, st, p);
    else hipLaunchKernelGGL(terms_prep_kernel<false>, grid, block, 0, st, p);
}

void launch_wgrad_terms(int bm, int bn, int grid, const WgradP &p, hipStream_t st)
{
    const dim3 g(grid), b(kConvThreads);
    if (bm == 128) hipLaunchKernelGGL((wgrad_terms_kernel<128, 64>), g, b, 0, st, p);
    else if (bn == 128) hipLaunchKernelGGL((wgrad_terms_kernel<64, 128>), g, b, 0, st, p);
    else hipLaunchKernelGGL((wgrad_terms_kernel<64, 64>), g, b, 0, st, p);
}

}  // namespace rn50
