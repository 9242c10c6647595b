// The network's first layer (3 input channels, 7x7, stride 2, pad 3, 64 filters) on the bf16 matrix instruction (device code; included
// by conv_stem.hip).  PREC 1: operands rounded to bf16, output / output gradient in bf16 (activations kept as bf16 in memory; the image is
// fp32).  PREC 2: fp32 operands split into three bf16 terms (see split8).
//
// Tiles, patch and persistent workgroups are those of stem_fwd_kernel: 8 x 16 output pixels, the 21 x 37 input pixels under them loaded
// once into LDS, coalesced, the next patch on its way while a tile is multiplied.  A patch row is stored without gaps: pixel
// (r, c) of the tile and element j of filter row fr sit at patch[(2r + fr) * kStemRowF + 6c + j].
#pragma once
#include <type_traits>

#include "conv_split.h"

namespace rn50 {

constexpr int kStemRowF = 116;   // a patch row: 111 elements, and what the last group of the last pixel reads beyond them (6*15 + 24)
constexpr int kStemGroups = 22;  // forward reduction: groups of 8 elements, three to a filter row (21 elements and three zeros), one of zeros
struct StemTile { int n, oh0, ow0; };
template <class P>
__device__ inline StemTile stem_tile(const P &p, int tile)
{
    const int n = tile / (p.tiles_h * p.tiles_w), rem = tile - n * (p.tiles_h * p.tiles_w), th = rem / p.tiles_w;
    return StemTile{n, th * kStemTH, (rem - th * p.tiles_w) * kStemTW};
}
template <class P>
__device__ __forceinline__ void stem_load_patch(const P &p, int tile, float (&v)[kStemLoads])
{
    const StemTile t = stem_tile(p, tile);
    const int ih0 = 2 * t.oh0 - 3, if0 = (2 * t.ow0 - 3) * 3;  // first input row; first float of the input rows
#pragma unroll
    for (int u = 0; u < kStemLoads; ++u) {
        const int i = (int)threadIdx.x + u * kConvThreads;
        const int pr = i / kStemCols, pc = i - pr * kStemCols;
        const int ih = ih0 + pr, f = if0 + pc;
        const bool ok = i < kStemRows * kStemCols && ih >= 0 && ih < p.IH && f >= 0 && f < p.IW * 3;
        v[u] = ok ? p.x[((long)t.n * p.IH + ih) * (p.IW * 3) + f] : 0.f;
    }
}
__device__ inline uint4 bf16_pack8(float4 a, float4 b) { return make_uint4(bf16_pack2(a.x, a.y), bf16_pack2(a.z, a.w), bf16_pack2(b.x, b.y), bf16_pack2(b.z, b.w)); }
__device__ inline floatx16 stem_mfma(uint4 a, uint4 b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Forward.  A lane's eight reduction elements are eight consecutive elements of a patch row, and the filter sits in LDS as the matrix
// instruction reads it.  STATS (whole tiles only): the tile's batch statistics as well.
// 32 x 224 x 224, split: 68 us with statistics (fp32 instruction 105, and 18 for the pass over the output); 256 x 224 x 224, bf16 output: 253 us with
// statistics where the general kernel's scalar gather took 853; writing 411 MB and reading 154 MB takes 120.
template <int PREC, bool STATS>
__global__ __launch_bounds__(kConvThreads, PREC == 2 ? 2 : 3) void stem_mm_fwd_kernel(StemMP p)
{
    constexpr bool SPLIT = PREC == 2;
    constexpr int NPL = SPLIT ? 3 : 1;
    __shared__ uint4 wl[NPL][kStemGroups * 64];
    __shared__ __attribute__((aligned(16))) float patch_mem[kStemRows * kStemRowF / (SPLIT ? 1 : 2)];
    __shared__ __attribute__((aligned(16))) uint16_t stage[SPLIT ? 8 : kStemTH * kStemTW * 64];
    __shared__ float s_mean[4][STATS ? 64 : 1], s_m2[4][STATS ? 64 : 1];
    float *patch = patch_mem;                                          // SPLIT
    uint16_t *patch16 = reinterpret_cast<uint16_t *>(patch_mem);       // else
    main_chain_priority();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < kStemGroups * 64; i += kConvThreads) {
        const int g = i >> 6, n = i & 63, fr = g / 3, j0 = 8 * (g % 3);
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = g < 21 && j0 + e < 21 ? p.w[n * 147 + fr * 21 + j0 + e] : 0.f;
        const float4 a = make_float4(v[0], v[1], v[2], v[3]), b = make_float4(v[4], v[5], v[6], v[7]);
        if (SPLIT) {
            const Split8 s = split8(a, b, split_up());
            wl[0][i] = s.hi;
            wl[NPL > 1 ? 1 : 0][i] = NPL > 1 ? s.mid : s.hi;
            wl[NPL > 2 ? 2 : 0][i] = NPL > 2 ? s.lo : s.hi;
        } else {
            wl[0][i] = bf16_pack8(a, b);
        }
    }
    for (int i = tid; i < (int)(sizeof(patch_mem) / 4); i += kConvThreads) patch_mem[i] = 0.f;  // what no load writes
    __syncthreads();

    const int pix = lane & 31, half = lane >> 5;
    const int tr = 2 * wave + (pix >> 4), tc = pix & 15;  // this lane's pixel of the tile, as the A operand's row
    const int abase = 2 * tr * kStemRowF + 6 * tc;
    const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
    float v[kStemLoads];
    if ((int)blockIdx.x < p.ntiles) stem_load_patch(p, blockIdx.x, v);
    for (int tile = blockIdx.x; tile < p.ntiles; tile += gridDim.x) {
        const StemTile t = stem_tile(p, tile);
        const float up = split_up();
#pragma unroll
        for (int u = 0; u < kStemLoads; ++u) {
            const int i = tid + u * kConvThreads;
            const int pr = i / kStemCols, pc = i - pr * kStemCols;
            if (i < kStemRows * kStemCols) {
                if (SPLIT) patch[pr * kStemRowF + pc] = v[u] * up;
                else patch16[pr * kStemRowF + pc] = (uint16_t)bf16_rne(v[u]);
            }
        }
        __syncthreads();
        if (tile + (int)gridDim.x < p.ntiles) stem_load_patch(p, tile + gridDim.x, v);

        floatx16 acc[2], accl[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = accl[j][e] = 0.f;
#pragma unroll
        for (int s = 0; s < kStemGroups / 2; ++s) {
            // lanes 0-31 take group 2s, lanes 32-63 group 2s+1; the last three elements of a filter row's third group are other pixels'
            const int ga = 2 * s, gb = 2 * s + 1;
            const int off = half ? (gb < 21 ? gb / 3 * kStemRowF + 8 * (gb % 3) : 0) : ga / 3 * kStemRowF + 8 * (ga % 3);
            const bool tail = half ? gb % 3 == 2 : ga % 3 == 2, none = half && gb == 21;
            uint4 ta[3];
            if (SPLIT) {
                const float2 *q = reinterpret_cast<const float2 *>(&patch[abase + off]);
                const float2 q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
                float4 lo = make_float4(q0.x, q0.y, q1.x, q1.y), hi = make_float4(q2.x, q2.y, q3.x, q3.y);
                if (tail) hi.y = hi.z = hi.w = 0.f;
                if (none) lo = hi = z4;
                const Split8 sp = split8_scaled(lo, hi);
                ta[0] = sp.hi; ta[1] = sp.mid; ta[2] = sp.lo;
            } else {
                const uint32_t *q = reinterpret_cast<const uint32_t *>(patch16) + ((abase + off) >> 1);
                uint4 a = make_uint4(q[0], q[1], q[2], q[3]);
                if (tail) {
                    a.z &= 0xffffu;
                    a.w = 0u;
                }
                if (none) a = make_uint4(0u, 0u, 0u, 0u);
                ta[0] = ta[1] = ta[2] = a;
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int wi = (ga + half) * 64 + j * 32 + pix;
                acc[j] = stem_mfma(ta[0], wl[0][wi], acc[j]);
                if (SPLIT) {
                    const uint4 bm = wl[NPL > 1 ? 1 : 0][wi], bl = wl[NPL > 2 ? 2 : 0][wi];
                    accl[j] = stem_mfma(ta[0], bm, accl[j]);
                    accl[j] = stem_mfma(ta[1], wl[0][wi], accl[j]);
                    accl[j] = stem_mfma(ta[1], bm, accl[j]);
                    accl[j] = stem_mfma(ta[0], bl, accl[j]);
                    accl[j] = stem_mfma(ta[2], wl[0][wi], accl[j]);
                }
            }
        }
        if (SPLIT) {
            bool bad = false;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    acc[j][e] = (acc[j][e] + accl[j][e]) * kSplitDown;
                    bad |= !isfinite(acc[j][e]);
                }
            if (__any(bad)) {  // an infinite operand has no finite split: this block on the fp32 instruction
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
#pragma clang loop unroll(disable)
                for (int k = 0; k < 7 * 11; ++k) {  // from memory: the patch holds scaled values
                    const int fr = k / 11, j = 2 * (k - fr * 11) + half;
                    const bool ok = j < 21;
                    const int ih = 2 * (t.oh0 + tr) - 3 + fr, f = (2 * (t.ow0 + tc) - 3) * 3 + j;
                    const float a = ok && ih >= 0 && ih < p.IH && f >= 0 && f < p.IW * 3 ? p.x[((long)t.n * p.IH + ih) * (p.IW * 3) + f] : 0.f;
                    const int wo = pix * 147 + fr * 21 + min(j, 20);
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, ok ? p.w[wo] : 0.f, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, ok ? p.w[wo + 32 * 147] : 0.f, acc[1], 0, 0, 0);
                }
            }
        }
        if (STATS) {  // of the tensor as stored; a wavefront's 32 pixels in two passes, the four wavefronts merged after Chan et al.
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float sum = 0.f, dev = 0.f;
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    if (!SPLIT) {
                        const uint32_t w = bf16_pack2(acc[j][e], acc[j][e + 1]);
                        acc[j][e] = bf16_lo(w);
                        acc[j][e + 1] = bf16_hi(w);
                    }
                    sum += acc[j][e];
                    sum += acc[j][e + 1];
                }
                sum += __shfl_xor(sum, 32, 64);
                const float mean = sum * (1.f / 32);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float d = acc[j][e] - mean;
                    dev = fmaf(d, d, dev);
                }
                dev += __shfl_xor(dev, 32, 64);
                if (lane < 32) {
                    s_mean[wave][j * 32 + lane] = mean;
                    s_m2[wave][j * 32 + lane] = dev;
                }
            }
            __syncthreads();  // the next write comes after the barrier at the end of the loop
            if (tid < 64) {
                float mean = s_mean[0][tid], m2 = s_m2[0][tid];
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    const float d = s_mean[w][tid] - mean;
                    mean = fmaf(d, 1.f / (w + 1), mean);
                    m2 += s_m2[w][tid] + d * d * (32.f * w / (w + 1));
                }
                p.mean[(size_t)tile * 64 + tid] = mean;
                p.m2[(size_t)tile * 64 + tid] = m2;
            }
        }
        // accumulator element e of lane l: row 8*(e/4) + 4*(l/32) + e%4 of the wavefront's 32 pixels, column l%32 of its block
        if (SPLIT) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int q = 8 * (e >> 2) + 4 * half + (e & 3);
                const int oh = t.oh0 + 2 * wave + (q >> 4), ow = t.ow0 + (q & 15);
                if (oh < p.OH && ow < p.OW) {
                    float *o = reinterpret_cast<float *>(p.y) + (((long)t.n * p.OH + oh) * p.OW + ow) * 64 + pix;
                    o[0] = acc[0][e];
                    o[32] = acc[1][e];
                }
            }
        } else {  // through LDS, 16 bytes per lane (see igemm_finish_act)
            uint16_t *st = stage + wave * (32 * 64);
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const int q = 8 * (e >> 2) + 4 * half + (e & 3);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint32_t w = bf16_pack2(acc[j][e], acc[j][e + 1]);
                    st[q * 64 + j * 32 + pix] = (uint16_t)w;
                    st[(q + 1) * 64 + j * 32 + pix] = (uint16_t)(w >> 16);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wavefront's own stores
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = u * 8 + (lane >> 3);
                const int oh = t.oh0 + 2 * wave + (q >> 4), ow = t.ow0 + (q & 15);
                const uint4 o = *reinterpret_cast<const uint4 *>(&st[q * 64 + (lane & 7) * 8]);
                if (oh < p.OH && ow < p.OW)
                    *reinterpret_cast<uint4 *>(reinterpret_cast<bf16_t *>(p.y) + (((long)t.n * p.OH + oh) * p.OW + ow) * 64 + (lane & 7) * 8) = o;
            }
        }
        __syncthreads();  // every wavefront is done with the patch before the next tile overwrites it
    }
}

// Filter gradient: dw[k][fr][j] = sum over output pixels of dy[pixel][k] * x[2*oh + fr - 3][(2*ow - 3)*3 + j], j = 0..20 the 7 taps x 3
// channels of a filter row, consecutive floats of an image row.  The product is [64 filters] x [128 pixels] x [147 -> 160 filter elements]: ten
// 32x32 blocks; a step of the matrix instruction is a row of 16 pixels.  Each wavefront takes two rows for all ten blocks (160
// accumulator registers) and keeps accumulating over every tile of the persistent workgroup, so the four wavefronts' sums meet
// only once, at the end, through LDS in wavefront order.  The workgroup leaves one partial [64][147]; the ordered sum over
// workgroups is splitk_reduce_kernel's.  With split operands all six products go into one accumulator, small ones first (two would need
// 320): six roundings per 16 pixels, where the fp32 instruction has eight.
// 32 x 224 x 224, split: 72 us (fp32 instruction 110): the splits of the gathered operand and the LDS reads under them, in four
// wavefronts that share an image tile.  256 x 224 x 224, bf16: 181 us with its reduction (general kernel 588).
template <int PREC>
__global__ __launch_bounds__(kConvThreads, 2) void stem_mm_wgrad_kernel(StemWP p)
{
    constexpr bool SPLIT = PREC == 2;
    constexpr int EPL = SPLIT ? 4 : 8, DYL = kStemTH * kStemTW * 64 / EPL / kConvThreads;  // elements and 16-byte loads of dy per thread and tile
    __shared__ __attribute__((aligned(16))) float patch[kStemRows * kStemRowF];
    __shared__ __attribute__((aligned(16))) float dyl[SPLIT ? kStemTH * kStemTW * 64 : 5 * 16 * 64];  // [pixel of the tile][filter]; the merge
    static_assert(5 * 16 * 64 * 4 >= kStemTH * kStemTW * 64 * 2, "the bf16 tile fits");
    uint16_t *dyh = reinterpret_cast<uint16_t *>(dyl);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    for (int i = tid; i < kStemRows * kStemRowF; i += kConvThreads) patch[i] = 0.f;  // the floats no load writes must not hold NaNs
    int cj[5];  // filter element 32*nb + col of this lane in block nb: its place in a patch relative to the pixel's
#pragma unroll
    for (int nb = 0; nb < 5; ++nb) {
        const int c = min(32 * nb + col, 146), fr = c / 21;
        cj[nb] = fr * kStemRowF + c - fr * 21;
    }
    const float sign = blockIdx.x & 1 ? -1.f : 1.f;  // SPLIT: every other workgroup multiplies with -dy and negates its
    // sums: a rounding of the instruction that prefers one direction cancels in the sum over workgroups (N = 32: error 7e-7 -> 3e-7)
    floatx16 acc[2][5];
    auto clear = [&]() {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int nb = 0; nb < 5; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[mb][nb][e] = 0.f;
    };
    auto run = [&](auto unit) {  // over all tiles of this workgroup; unit: on the fp32 instruction
        constexpr bool UNIT = decltype(unit)::value;
        clear();
        for (int tile = blockIdx.x; tile < p.ntiles; tile += gridDim.x) {
            const StemTile t = stem_tile(p, tile);
            float v[kStemLoads];
            uint4 g[DYL];
            stem_load_patch(p, tile, v);
#pragma unroll
            for (int u = 0; u < DYL; ++u) {
                const int i = tid + u * kConvThreads;  // 16-byte index: 64 / EPL of them to a pixel
                const int q = i / (64 / EPL), oh = t.oh0 + (q >> 4), ow = t.ow0 + (q & 15);
                // a pixel outside the output contributes nothing: its dy is zero (the patch under it holds zeros or other pixels' values, see below)
                const char *src = reinterpret_cast<const char *>(p.dy) + ((((long)t.n * p.OH + oh) * p.OW + ow) * 64 + EPL * (i % (64 / EPL))) * (16 / EPL);
                g[u] = (oh < p.OH && ow < p.OW) ? *reinterpret_cast<const uint4 *>(src) : make_uint4(0u, 0u, 0u, 0u);
            }
            __syncthreads();  // every wavefront is done with the previous tile
            constexpr bool SCALED = SPLIT && !UNIT;
            const float up = split_up(), upg = sign * up;
#pragma unroll
            for (int u = 0; u < kStemLoads; ++u) {
                const int i = tid + u * kConvThreads;
                const int pr = i / kStemCols, pc = i - pr * kStemCols;
                if (i < kStemRows * kStemCols) patch[pr * kStemRowF + pc] = SCALED ? v[u] * up : v[u];
            }
#pragma unroll
            for (int u = 0; u < DYL; ++u) {
                if (SCALED) g[u] = __builtin_bit_cast(uint4, scaled4(__builtin_bit_cast(float4, g[u]), upg));
                reinterpret_cast<uint4 *>(dyl)[tid + u * kConvThreads] = g[u];
            }
            __syncthreads();
            if (UNIT) {
#pragma clang loop unroll(disable)
                for (int s = 0; s < 16; ++s) {  // pixel pairs: lane half h multiplies pixel 2s + h of this wavefront's 32
                    const int q = 32 * wave + 2 * s + half;
                    const int pb = 2 * (q >> 4) * kStemRowF + 6 * (q & 15);
                    const float a0 = dyl[q * 64 + col], a1 = dyl[q * 64 + 32 + col];
#pragma unroll
                    for (int nb = 0; nb < 5; ++nb) {
                        const float b = patch[pb + cj[nb]];
                        acc[0][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b, acc[0][nb], 0, 0, 0);
                        acc[1][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b, acc[1][nb], 0, 0, 0);
                    }
                }
                continue;
            }
#pragma clang loop unroll(disable)
            for (int rr = 0; rr < 2; ++rr) {
                const int r = 2 * wave + rr;
                uint4 ta[2][3];
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    if (SPLIT) {
                        const float *q = &dyl[(r * 16 + 8 * half) * 64 + mb * 32 + col];
                        const Split8 s = split8_scaled(make_float4(q[0], q[64], q[128], q[192]), make_float4(q[256], q[320], q[384], q[448]));
                        ta[mb][0] = s.hi; ta[mb][1] = s.mid; ta[mb][2] = s.lo;
                    } else {  // transposing reads, as in wgrad_act_copy_kernel
                        const uint16_t *q = &dyh[(r * 16 + 8 * half + ((lane & 15) >> 2)) * 64 + mb * 32 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4];
                        ta[mb][0] = ta[mb][1] = ta[mb][2] = __builtin_bit_cast(uint4, Frag8{lds_read_tr(q), lds_read_tr(q + 4 * 64)});
                    }
                }
#pragma unroll
                for (int nb = 0; nb < 5; ++nb) {
                    const float *q = &patch[2 * r * kStemRowF + 48 * half + cj[nb]];
                    const float4 lo = make_float4(q[0], q[6], q[12], q[18]), hi = make_float4(q[24], q[30], q[36], q[42]);
                    if (SPLIT) {
                        const Split8 s = split8_scaled(lo, hi);
                        const uint4 tb[3] = {s.hi, s.mid, s.lo};
                        constexpr int ia[6] = {0, 2, 1, 0, 1, 0}, ib[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
                        for (int pr = 0; pr < 6; ++pr)
#pragma unroll
                            for (int mb = 0; mb < 2; ++mb) acc[mb][nb] = stem_mfma(ta[mb][ia[pr]], tb[ib[pr]], acc[mb][nb]);
                    } else {
                        const uint4 b = bf16_pack8(lo, hi);
#pragma unroll
                        for (int mb = 0; mb < 2; ++mb) acc[mb][nb] = stem_mfma(ta[mb][0], b, acc[mb][nb]);
                    }
                }
            }
        }
    };
    run(std::integral_constant<bool, false>());
    if (SPLIT) {
        bool bad = false;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int nb = 0; nb < 5; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    acc[mb][nb][e] *= sign * kSplitDown;
                    bad |= !isfinite(acc[mb][nb][e]);
                }
        if (__syncthreads_or(bad)) run(std::integral_constant<bool, SPLIT>());  // an infinite operand has no finite split: all again on the fp32 instruction
    }
    // the four wavefronts' sums, added in wavefront order through LDS, one half of the filters at a time (5 x 16 x 64 floats = 20 KB)
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
        for (int w = 1; w < 4; ++w) {
            __syncthreads();
            if (wave == w) {
#pragma unroll
                for (int nb = 0; nb < 5; ++nb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) dyl[(nb * 16 + e) * 64 + lane] = acc[mb][nb][e];
            }
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int nb = 0; nb < 5; ++nb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[mb][nb][e] += dyl[(nb * 16 + e) * 64 + lane];
            }
        }
    if (wave == 0) {
        float *out = p.part + (long)blockIdx.x * (64 * 147);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int nb = 0; nb < 5; ++nb) {
                const int c = 32 * nb + col;
                if (c < 147) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) out[(32 * mb + 8 * (e >> 2) + 4 * half + (e & 3)) * 147 + c] = acc[mb][nb][e];
                }
            }
    }
}

}  // namespace rn50
