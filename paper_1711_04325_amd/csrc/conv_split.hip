// Launches of the kernels of conv_split.h.
#include "conv_split.h"

namespace rn50 {

size_t filter_planes_bytes(int rows, int kdim) { return (size_t)(kdim / kBK) * plane_rows_of(rows) * kPlaneRow; }

void launch_filter_split(int rows, int kdim, const float *w, char *planes, hipStream_t st)
{
    SplitJob job{};
    job.rows = rows;
    job.plane_rows = plane_rows_of(rows);
    job.kdim = kdim;
    hipLaunchKernelGGL(filter_split_kernel, dim3(split_job_blocks(rows, kdim)), dim3(256), 0, st, job, w, planes);
}

void launch_filter_split_batched(const void *jobs, int njobs, int nblocks, const float *base, char *planes, hipStream_t st)
{
    hipLaunchKernelGGL(filter_split_batched_kernel, dim3(nblocks), dim3(256), 0, st, (const SplitJob *)jobs, njobs, base, planes);
}

template <int BM, int BN>
static void launch_pre(const IgemmP &p, int grid, hipStream_t st)
{
    const dim3 g(grid), b(kConvThreads);
    if (p.sd > 1) hipLaunchKernelGGL((igemm_pre_kernel<BM, BN, 1, false, false>), g, b, 0, st, p);
    else if (p.in_scale && p.stat_mean) hipLaunchKernelGGL((igemm_pre_kernel<BM, BN, 0, true, true>), g, b, 0, st, p);
    else if (p.in_scale) hipLaunchKernelGGL((igemm_pre_kernel<BM, BN, 0, true, false>), g, b, 0, st, p);
    else if (p.stat_mean) hipLaunchKernelGGL((igemm_pre_kernel<BM, BN, 0, false, true>), g, b, 0, st, p);
    else hipLaunchKernelGGL((igemm_pre_kernel<BM, BN, 0, false, false>), g, b, 0, st, p);
}
void launch_igemm_pre(int bm, int bn, int grid, const IgemmP &p, hipStream_t st)
{
    if (bm == 128 && bn == 128) launch_pre<128, 128>(p, grid, st);
    else if (bm == 128) launch_pre<128, 64>(p, grid, st);
    else if (bn == 128) launch_pre<64, 128>(p, grid, st);
    else launch_pre<64, 64>(p, grid, st);
}

template <int BN, int WMAX>
static void launch_c3(const IgemmP &p, int grid, hipStream_t st)
{
    const dim3 g(grid), b(kConvThreads);
    if (p.in_scale && p.stat_mean) hipLaunchKernelGGL((conv3x3_kernel<128, BN, WMAX, true, true>), g, b, 0, st, p);
    else if (p.in_scale) hipLaunchKernelGGL((conv3x3_kernel<128, BN, WMAX, true, false>), g, b, 0, st, p);
    else if (p.stat_mean) hipLaunchKernelGGL((conv3x3_kernel<128, BN, WMAX, false, true>), g, b, 0, st, p);
    else hipLaunchKernelGGL((conv3x3_kernel<128, BN, WMAX, false, false>), g, b, 0, st, p);
}
void launch_conv3x3(int bn, int grid, const IgemmP &p, hipStream_t st)
{
    if (bn == 128) launch_c3<128, 28>(p, grid, st);
    else if (p.IW <= 28) launch_c3<64, 28>(p, grid, st);
    else launch_c3<64, 56>(p, grid, st);
}

}  // namespace rn50
