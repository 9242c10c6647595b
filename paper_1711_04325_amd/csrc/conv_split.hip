// Launches of the kernels of conv_split.h and conv_act.h.
#include "conv_act.h"

namespace rn50 {

size_t filter_planes_bytes(int rows, int kdim, bool act)
{
    return act ? (size_t)(kdim / kActBK) * plane_rows_of(rows) * kActRow : (size_t)(kdim / kBK) * plane_rows_of(rows) * kPlaneRow;
}

// one thread per 16-byte chunk of a plane: eight elements
int split_job_blocks(int rows, int kdim) { return ceil_div((long)plane_rows_of(rows) * (kdim / kBK) * 4, 256); }

SplitJobHost split_job(int rows, int kdim, long src_off, long dst_off, int block_begin)
{
    return SplitJobHost{src_off, dst_off, rows, plane_rows_of(rows), kdim, block_begin};
}

void launch_filter_planes(int rows, int kdim, bool act, const float *w, char *planes, hipStream_t st)
{
    const SplitJob job = split_job(rows, kdim, 0, 0, 0);
    const dim3 grid(split_job_blocks(rows, kdim)), block(256);
    if (act) hipLaunchKernelGGL(filter_round_kernel, grid, block, 0, st, job, w, planes);
    else hipLaunchKernelGGL(filter_split_kernel, grid, block, 0, st, job, w, planes);
}

void launch_filter_planes_batched(const void *jobs, int njobs, int nblocks, bool act, const float *base, char *planes, hipStream_t st)
{
    if (act) hipLaunchKernelGGL(filter_round_batched_kernel, dim3(nblocks), dim3(256), 0, st, (const SplitJob *)jobs, njobs, base, planes);
    else hipLaunchKernelGGL(filter_split_batched_kernel, dim3(nblocks), dim3(256), 0, st, (const SplitJob *)jobs, njobs, base, planes);
}

template <int BM, int BN>
static void launch_pre(const IgemmP &p, int grid, hipStream_t st)
{
    const dim3 g(grid), b(kConvThreads);
    if constexpr (BM == 64) {
        if (p.sd > 1) {
            hipLaunchKernelGGL((igemm_pre_kernel<BM, BN, 1, false, false>), g, b, 0, st, p);
            return;
        }
    }
    if (p.in_scale && p.stat_mean) hipLaunchKernelGGL((igemm_pre_kernel<BM, BN, 0, true, true>), g, b, 0, st, p);
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

template <int BM, int BN>
static void launch_act(const IgemmP &p, int grid, hipStream_t st)
{
    const dim3 g(grid), b(kConvThreads);
    if (p.sd > 1) hipLaunchKernelGGL((igemm_act_kernel<BM, BN, 1, false>), g, b, 0, st, p);
    else if (p.stat_mean) hipLaunchKernelGGL((igemm_act_kernel<BM, BN, 0, true>), g, b, 0, st, p);
    else hipLaunchKernelGGL((igemm_act_kernel<BM, BN, 0, false>), g, b, 0, st, p);
}
void launch_igemm_act(int bm, int bn, int grid, const IgemmP &p, hipStream_t st)
{
    if (bm == 128 && bn == 128) launch_act<128, 128>(p, grid, st);
    else if (bm == 128) launch_act<128, 64>(p, grid, st);
    else if (bn == 128) launch_act<64, 128>(p, grid, st);
    else launch_act<64, 64>(p, grid, st);
}

template <int BM, int BN>
static void launch_wgrad_copy(const WgradP &p, int grid, hipStream_t st)
{
    if (p.in_scale) hipLaunchKernelGGL((wgrad_act_copy_kernel<BM, BN, true>), dim3(grid), dim3(kConvThreads), 0, st, p);
    else hipLaunchKernelGGL((wgrad_act_copy_kernel<BM, BN, false>), dim3(grid), dim3(kConvThreads), 0, st, p);
}
void launch_wgrad_act_copy(int bm, int bn, int grid, const WgradP &p, hipStream_t st)
{
    if (bm == 128 && bn == 128) launch_wgrad_copy<128, 128>(p, grid, st);
    else if (bm == 128) launch_wgrad_copy<128, 64>(p, grid, st);
    else if (bn == 128) launch_wgrad_copy<64, 128>(p, grid, st);
    else launch_wgrad_copy<64, 64>(p, grid, st);
}

template <int BM, int BN>
static void launch_wgrad(const WgradP &p, int grid, hipStream_t st)
{
    if (p.in_scale) hipLaunchKernelGGL((wgrad_split_kernel<BM, BN, true>), dim3(grid), dim3(kConvThreads), 0, st, p);
    else hipLaunchKernelGGL((wgrad_split_kernel<BM, BN, false>), dim3(grid), dim3(kConvThreads), 0, st, p);
}
void launch_wgrad_split(int bm, int bn, int grid, const WgradP &p, hipStream_t st)
{
    if (bm == 128 && bn == 128) launch_wgrad<128, 128>(p, grid, st);
    else if (bm == 128) launch_wgrad<128, 64>(p, grid, st);
    else if (bn == 128) launch_wgrad<64, 128>(p, grid, st);
    else launch_wgrad<64, 64>(p, grid, st);
}

}  // namespace rn50
