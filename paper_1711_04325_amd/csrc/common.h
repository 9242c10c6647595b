// Internal helpers shared by the translation units of librn50.so (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include <memory>
#include <vector>

#include "rn50.h"

namespace rn50 {

int fail(int code, const char *fmt, ...);  // records the message for rn50_last_error() and returns code

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// After a kernel launch: turn a launch error into RN50_EHIP.
inline int launch_status(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RN50_EHIP, "%s: %s", what, hipGetErrorString(e));
    return RN50_OK;
}

// Tuning and test switches (rn50_set_option; initial values from the RN50_* environment variables, read once).
struct PlanRow { int op, n, c, h, k, r, stride, pad, bm, bn, split; };
struct Config {
    bool side_stream = true;   // rn50_create: filter gradients and projection shortcuts on helper streams
    int fuse_bn = -1;          // rn50_create: which BN + ReLU outputs are applied by their consumer (bit mask); -1: 3, with bf16 activations 1
    bool relu_mask = true;     // rn50_create: byte mask instead of the block output in the c layers' BN backward
    bool no_tuned = false;     // ignore the measured plan table (cost model only)
    bool no_stem_kernel = false;  // first layer through the implicit GEMM
    bool split_products = false;  // rn50_create: the training step's forward pass with split operands as well
    int half_products = 3;        // calls with fp32 operands that may choose fp16 halves: 1 forward, 2 data gradients
    bool conv_bn_stats = true;    // rn50_create: forward convolutions gather the BN statistics of their output
    int wgrad_group = 0;          // rn50_create: filter gradients launched per layer (0) or grouped, this many blocks to a launch
    int wgrad_group_wgs_per_cu = 0;  // grouped filter gradients: at most this many workgroups of theirs per CU (0: what fits)
    int wgrad_group_stages = 48;  // grouped filter gradients: LDS stages (of 32 pixels) per work item
    int wgrad_group_bm = 64, wgrad_group_bn = 64;  // ... and their tile
    bool has_igemm_plan = false, has_wgrad_plan = false;
    int igemm_plan[3] = {0, 0, 0}, wgrad_plan[3] = {0, 0, 0};  // bm, bn, split forced for every call
    std::vector<PlanRow> pre_plans;                            // plans of the calls whose filter is prepared beforehand
    std::vector<PlanRow> operand_plans;                        // plans of calls that prepare both operands, which their call then does
    std::vector<PlanRow> small_plans;                          // plans of igemm_small_kernel (tiles of 16 or 32; the cut says nothing)
    std::vector<PlanRow> overrides;                            // rows that go before the measured table
};
std::shared_ptr<const Config> config();  // the current snapshot (immutable), or the one that this thread's ConfigScope holds
// A call of the ABI holds the snapshot it started with, whatever other threads set meanwhile: it plans more than once (what to
// prepare, how much room, what to launch), and the decisions have to be those of one plan.
class ConfigScope {
public:
    ConfigScope();
    ~ConfigScope();
    ConfigScope(const ConfigScope &) = delete;
    ConfigScope &operator=(const ConfigScope &) = delete;

private:
    std::shared_ptr<const Config> held;
    bool outermost;
};

inline int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }

constexpr int kWave = 64;

// Sum over the 64 lanes of a wavefront (result valid in every lane).
__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ inline float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// ---- activation storage: fp32, or bfloat16 bits (round to nearest even on store) ------------------------------------
typedef uint16_t bf16_t;

// fp32 -> bfloat16 bits, round to nearest, ties to even (NaN stays NaN): gfx950 converts in hardware, two values per
// instruction (v_cvt_pk_bf16_f32); in integer arithmetic the same rounding costs about five instructions per value, in
// kernels that round every operand on its way into LDS.  A conversion that the compiler knows: it keeps the wait states
// that the hardware wants between it and a matrix instruction, whose operand it makes (2) or whose result it reads (up to
// 20).  Around inline assembly it counts none.
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t bf16_pack2(float lo, float hi)
{
    const floatx2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// The same as the bare instruction, for values in registers that neither come from a matrix instruction nor go to one: the
// filter-gradient kernels pair elements of two register arrays, and building a vector of those makes the compiler keep the
// arrays in scratch memory.
__device__ inline uint32_t bf16_pack2_bare(float lo, float hi)
{
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(lo), "v"(hi));
    return r;
}
__device__ inline uint32_t bf16_rne(float f) { return bf16_pack2(f, f) & 0xffffu; }
__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }          // element in the low half of a word
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }  // element in the high half
__device__ inline float bf16_round(float f) { return __uint_as_float(bf16_rne(f) << 16); }

// Elements 4*i4 .. 4*i4+3 of a tensor as floats, and the store of four floats (the bf16 store rounds).
__device__ inline float4 ld4(const float *p, size_t i4) { return reinterpret_cast<const float4 *>(p)[i4]; }
__device__ inline float4 ld4(const bf16_t *p, size_t i4)
{
    const uint2 u = reinterpret_cast<const uint2 *>(p)[i4];
    return make_float4(bf16_lo(u.x), bf16_hi(u.x), bf16_lo(u.y), bf16_hi(u.y));
}
__device__ inline void st4(float *p, size_t i4, float4 v) { reinterpret_cast<float4 *>(p)[i4] = v; }
__device__ inline void st4(bf16_t *p, size_t i4, float4 v)
{
    reinterpret_cast<uint2 *>(p)[i4] = make_uint2(bf16_pack2(v.x, v.y), bf16_pack2(v.z, v.w));
}
// What a store of v leaves in memory, as floats (the forward output's sign decides the ReLU mask: it is taken after rounding).
__device__ inline float4 as_stored(const float *, float4 v) { return v; }
__device__ inline float4 as_stored(const bf16_t *, float4 v) { return make_float4(bf16_round(v.x), bf16_round(v.y), bf16_round(v.z), bf16_round(v.w)); }

// Issue priority of the calling wavefront among the wavefronts of its SIMD (0 = default = lowest, 3 = highest); see igemm_kernel.
__device__ inline void main_chain_priority() { __builtin_amdgcn_s_setprio(3); }

// Consecutive workgroups are dispatched to different XCDs, each with an L2 of its own.  Workgroup b of n does the work of
// index xcd_contiguous(b, n): the eight XCDs then each cover one contiguous range of the index space, so that neighbouring
// work items, which read the same cache lines, share an L2.
__device__ inline int xcd_contiguous(int b, int n)
{
    const int n8 = n & ~7;
    return b < n8 ? (b & 7) * (n8 >> 3) + (b >> 3) : b;
}

}  // namespace rn50

namespace rn50 {
// Internal entry points used by the whole-step schedule (csrc/conv.hip).
int conv_check(const char *who, const rn50_conv_desc *d);  // argument checks shared by the convolution entry points
// How products of fp32 operands are formed.  kFp32Split: operands split into bf16 terms (see split8 in conv_kernels.h; every call
// of the ABI that has the workspace its query names).  kFp32Unit: the fp32 matrix instruction, with the
// tiles, pieces and order of sums of the measured table (the forward pass of a training context: see rn50_ctx).
// kNoHalf: kFp32Split without the kernels on fp16 halves (conv_half.h).
// kNoPlanes: the fp32 instruction, and with bf16 activations the kernels that take the filter as it is (a call with less workspace).
enum Fp32Math { kFp32Unit, kFp32Split, kNoHalf, kNoPlanes };
size_t conv_workspace(const rn50_conv_desc *d, int op, Fp32Math math, bool given);  // rn50_conv_workspace_bytes; given: with `planes`
// `planes`: the call's filter prepared beforehand by launch_filter_planes_batched (null: the call does it where its kernel wants it
// so); conv_planes_bytes says how much room it takes (0: the kernel of this call takes none), for op RN50_OP_FWD or RN50_OP_BWD_DATA.
size_t conv_planes_bytes(const rn50_conv_desc *d, int op);
int conv_fwd_math(Fp32Math math, const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift, const float *w,
                  const char *planes, float *y, void *ws, size_t ws_bytes, hipStream_t st);
// The forward pass followed by z = y*scale[c] + shift[c] [+ residual] [ReLU] (fp32 storage, K % 4 == 0).
int conv_fwd_apply_math(Fp32Math math, const rn50_conv_desc *d, const float *x, const float *w, const char *planes, float *y, const float *scale,
                        const float *shift, const float *residual, int relu, float *z, void *ws, size_t ws_bytes, hipStream_t st);
int conv_fwd_bnstats_math(Fp32Math math, const rn50_conv_desc *d, const float *x, const float *in_scale_or_null, const float *in_shift_or_null,
                          const float *w, const char *planes, float *y, const float *gamma, const float *beta, float eps, float *save_mean,
                          float *save_invstd, float *scale, float *shift, void *ws, size_t ws_bytes, hipStream_t st);
int conv_bwd_data_pretransposed(Fp32Math math, const rn50_conv_desc *d, const float *dy, const float *wt, float *dx, void *ws, size_t ws_bytes,
                                hipStream_t st, const char *planes = nullptr, bool flipped = true);
int conv_bwd_weight_math(Fp32Math math, const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift, const float *dy,
                         float *dw, void *ws, size_t ws_bytes, hipStream_t st);
void launch_filter_flip(int K, int C, int RS, const float *w, float *wt, hipStream_t st);
// One launch for many filters; `jobs` is a device array of FlipJobHost records (same layout as the kernel's).
struct FlipJobHost {
    int K, C, RS, tiles_c, tiles_k, block_begin;
    long src_off, dst_off;
};
// The same for the preparation of many filters (csrc/conv_split.hip; split into bf16 terms, or with act rounded to bf16): filter j has `rows` rows of `kdim` elements at src_off (elements from the
// launch's base) and its planes at dst_off (bytes).
struct SplitJobHost {
    long src_off, dst_off;
    int rows, plane_rows, kdim, block_begin;
};
SplitJobHost split_job(int rows, int kdim, long src_off, long dst_off, int block_begin);
int split_job_blocks(int rows, int kdim);
void launch_filter_planes_batched(const void *jobs, int njobs, int nblocks, bool act, const float *base, char *planes, hipStream_t st);
// Scale and shift of many BN layers from given statistics (csrc/bn.hip), in one launch: layer j has `c` channels, its gamma and beta at
// g_off and b_off elements of theta, its mean, 1/sigma, scale and shift at byte offsets of `arena`.
struct BnLayerHost {
    long g_off, b_off, mean, invstd, scale, shift;
    int c, pad_;
};
void launch_bn_scale_shift_batched(const void *layers, int n, int max_c, const float *theta, char *arena, hipStream_t st);
// y = x*scale[c] + shift[c] [ReLU] over an N x H x W x C tensor (the normalising kernel of the BN forward alone).
int bn_apply_scale_shift(int n, int c, int h, int w, const float *x, const float *scale, const float *shift, int relu, float *y,
                         hipStream_t st);
int bn_apply_scale_shift_bf16(int n, int c, int h, int w, const uint16_t *x, const float *scale, const float *shift, int relu,
                              uint16_t *y, hipStream_t st);
// Merge of per-row-tile statistics gathered by a convolution: `bands` tiles of rows_per_band rows each (the last one
// ragged) left mean and squared deviations at part_mean / part_m2 [band][C]; writes what the BN forward's merge writes.
// fold: many partials are merged in two launches (another order of the sums).
void bn_finalize_partials(bool fold, long M, int C, int bands, int rows_per_band, float *part_mean, float *part_m2,
                          const float *gamma, const float *beta, float eps, float *save_mean, float *save_invstd, float *scale,
                          float *shift, hipStream_t st);
// Filter gradients of several layers in one launch (csrc/conv_group.hip): the extern "C" calls with the tuning values spelled out.
size_t wgrad_group_table_bytes(int count);
size_t wgrad_group_ws_bytes(int count, const rn50_wgrad_group_item *items, int stages);
int wgrad_group_plan(int count, const rn50_wgrad_group_item *items, void *ws, size_t ws_bytes, void *table_host, size_t table_bytes,
                     int stages, int bm, int bn, int wgs_per_cu);
constexpr int kFlipTileHost = 64;  // tile edge of the filter flip kernels (a job counts its workgroups with it)
void launch_filter_flip_batched(const void *jobs, int njobs, int nblocks, const float *theta, float *wt, hipStream_t st);
}  // namespace rn50

#define RN50_REQUIRE(cond, code, ...) \
    do { if (!(cond)) return rn50::fail(code, __VA_ARGS__); } while (0)
