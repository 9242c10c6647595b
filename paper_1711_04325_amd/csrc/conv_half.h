// fp32 products as three fp16 ones (device code; included by conv_half.hip).
//
// An fp32 number x, multiplied by a power of two that brings the largest finite number of its tensor into [2^14, 2^15), is hi + lo *
// 2^-12 with hi the nearest fp16 number and lo the nearest one to 2^12 times the rest: 22 to 24 bits.  Of the four products of two such
// numbers hi*hi, hi*lo and lo*hi are formed; lo*lo is below 2^-22 of the product.  The chip is bound by its power in long sums of
// products: with operands of random bits a loop of nothing but v_mfma_f32_32x32x16_bf16 runs at 1.8 GHz instead of 2.4, 302 TFLOP/s of
// six-product fp32 work (278 with its LDS reads), and three v_mfma_f32_16x16x32_f16 reach 654 (576; with v_mfma_f32_32x32x16_f16 569 and
// 518: the same bits, more power).
//
// Error against 64 bits (relative 2-norm, normal operands / behind a ReLU, reduction of 512, 1152, 2304, 4608): six bf16 products
// 1.3e-7, 2.0e-7, 2.9e-7, 4.2e-7 / 1.0e-7, 1.6e-7, 2.3e-7, 3.5e-7; here 1.2e-7, 1.2e-7, 1.4e-7, 1.6e-7 / 1.2e-7, 1.3e-7, 1.4e-7,
// 1.6e-7: the sums of hi*hi are moved to accumulators of their own every 128 elements (without that 1.7e-7 .. 4.4e-7).  What stays, 9e-8, are the
// bits that the halves drop: so sums of 700 products and more come here, of 480 in data gradients (half_as_precise in conv.hip).
//
// The fixed range: numbers below 2^-27 of their tensor's largest one have fewer than 24 bits, below 2^-52 none.  Beside larger ones that is
// nothing where those meet weights like the others', but not where theirs are zero or as small as the numbers are large (channels with scales
// of their own).  So the split counts such numbers by place (32 pixels, or a filter row), and a wavefront forms its outputs again on the fp32
// instruction where one of them has no sum large enough to hide what the numbers under its block may have lost (kHalfFloor), as it does with
// results that are not finite.
#pragma once
#include "conv_terms.h"

namespace rn50 {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kHalfTop = 14;                 // exponent that the largest number gets
constexpr int kHalfLow = 12;                 // lo is kept times 2^12
constexpr float kHalfSmall = 0x1p-12f;       // numbers below this (and not zero) lose bits
constexpr float kHalfFloor = 16.f;           // sums above this for each of them hide what they lose: see igemm_half_kernel
constexpr int kHalfZeros = 256;               // zero bytes ahead of the gathered tensor's halves
constexpr int kHalfFlush = 4;                // stages of 32 between two moves of the hi*hi sums

__device__ inline unsigned finite_bits(float v)  // magnitude as an ordered integer; infinities and NaNs count as nothing
{
    const unsigned u = __float_as_uint(v) & 0x7fffffffu;
    return u < 0x7f800000u ? u : 0u;
}
// power of two by which a tensor with this largest magnitude is multiplied
__device__ inline int half_exponent(unsigned top)
{
    if (!top) return 0;
    int e;
    (void)frexpf(__uint_as_float(top), &e);  // top = f * 2^e, f in [0.5, 1)
    return kHalfTop + 1 - e;
}
struct Half8 { uint4 hi, lo; };
__device__ inline uint32_t half_pair(float x, float y, uint32_t &low)
{
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    const f16x2 h = {(_Float16)x, (_Float16)y};
    const f16x2 l = {(_Float16)((x - (float)h[0]) * (float)(1 << kHalfLow)), (_Float16)((y - (float)h[1]) * (float)(1 << kHalfLow))};
    low = __builtin_bit_cast(uint32_t, l);
    return __builtin_bit_cast(uint32_t, h);
}
__device__ inline Half8 half8(float4 a, float4 b)  // of scaled numbers
{
    Half8 r;
    r.hi.x = half_pair(a.x, a.y, r.lo.x);
    r.hi.y = half_pair(a.z, a.w, r.lo.y);
    r.hi.z = half_pair(b.x, b.y, r.lo.z);
    r.hi.w = half_pair(b.z, b.w, r.lo.w);
    return r;
}
__device__ inline float4 ldexp4(float4 v, int e) { return make_float4(ldexpf(v.x, e), ldexpf(v.y, e), ldexpf(v.z, e), ldexpf(v.w, e)); }
// how many of these numbers are not zero and, scaled, too small for the halves to hold their bits
__device__ inline unsigned tiny1(float v, float scaled) { return v != 0.f && fabsf(scaled) < kHalfSmall; }
__device__ inline unsigned tiny4(float4 v, float4 scaled) { return tiny1(v.x, scaled.x) + tiny1(v.y, scaled.y) + tiny1(v.z, scaled.z) + tiny1(v.w, scaled.w); }

// ---- preparation: two launches for both operands of a call -----------------------------------------------------------------
// First: the largest finite magnitude of each workgroup's share; marks cleared.
template <bool INAFF>
static __global__ __launch_bounds__(256) void half_max_kernel(HalfPrep p)
{
    __shared__ unsigned red[4];
    const int tid = threadIdx.x;
    for (int i = blockIdx.x * 256 + tid; i < p.nmarks; i += gridDim.x * 256) p.marks[i] = 0u;
    if (blockIdx.x == 0 && tid < kHalfZeros / 16) reinterpret_cast<uint4 *>(p.op[0].dst)[tid] = make_uint4(0u, 0u, 0u, 0u);  // ahead of the gathered tensor
    const int which = (int)blockIdx.x >= p.op[0].blocks;
    const HalfOperand &o = p.op[which];
    const int b = (int)blockIdx.x - (which ? p.op[0].blocks : 0);
    uint4 tops = make_uint4(0u, 0u, 0u, 0u);
    auto take = [&](unsigned i, float4 v) {
        if (INAFF && !which) {
            const unsigned c4 = i - fdiv(i, p.div_c4) * p.div_c4.d;
            v = bn_relu4(v, ldg4(p.in_scale + 4 * c4), ldg4(p.in_shift + 4 * c4));
        }
        tops.x = max(tops.x, finite_bits(v.x));
        tops.y = max(tops.y, finite_bits(v.y));
        tops.z = max(tops.z, finite_bits(v.z));
        tops.w = max(tops.w, finite_bits(v.w));
    };
    const unsigned step = (unsigned)o.blocks * 256u, n4 = o.n4;
    unsigned i = (unsigned)b * 256u + tid;
    const float4 *src = reinterpret_cast<const float4 *>(o.src);
    for (; i < n4 && n4 - i > 3 * step; i += 4 * step) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = src[i + u * step];
#pragma unroll
        for (int u = 0; u < 4; ++u) take(i + u * step, v[u]);
    }
    for (; i < n4; i += step) take(i, src[i]);
    unsigned top = max(max(tops.x, tops.y), max(tops.z, tops.w));
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) top = max(top, (unsigned)__shfl_xor((int)top, d, 64));
    if ((tid & 63) == 0) red[tid >> 6] = top;
    __syncthreads();
    if (tid == 0) o.part[b] = max(max(red[0], red[1]), max(red[2], red[3]));
}

// the tensor's largest magnitude from the shares; uniform over the workgroup
__device__ inline int half_up(const HalfOperand &o, unsigned *red)
{
    const int tid = threadIdx.x;
    unsigned top = 0;
    for (int i = tid; i < o.blocks; i += 256) top = max(top, o.part[i]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) top = max(top, (unsigned)__shfl_xor((int)top, d, 64));
    if ((tid & 63) == 0) red[tid >> 6] = top;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(half_exponent(max(max(red[0], red[1]), max(red[2], red[3]))));
}

// Second: the halves.  Tensors of pixels ([pixel][C], C % 32 == 0) as [pixel][C/32][hi of 32, lo of 32]; filters as [stage of 32][plane_rows][the
// same 128 bytes in the order of the LDS image], from [row][kdim], or flipped and transposed from [kdim / taps][taps][row].  One thread per eight elements.
template <bool INAFF>
static __global__ __launch_bounds__(256) void half_split_kernel(HalfPrep p)
{
    __shared__ unsigned red[4];
    const int tid = threadIdx.x;
    const int which = (int)blockIdx.x >= p.op[0].split_blocks;
    const HalfOperand &o = p.op[which];
    const int b = (int)blockIdx.x - (which ? p.op[0].split_blocks : 0);
    const int up = half_up(o, red);
    if (b == 0 && tid == 0) *o.up = up;
    for (unsigned i = (unsigned)b * 256u + tid; i < o.n8; i += (unsigned)o.split_blocks * 256u) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), c = a;
        uint4 *hi;
        unsigned *mark;
        int low_at = 4;  // the lo part's place, in 16-byte pieces from hi
        if (o.kind == kHalfPixels) {
            const unsigned pix = fdiv(i, o.div8), c8 = i - pix * o.div8.d;
            const float4 *s = reinterpret_cast<const float4 *>(o.src) + 2 * (size_t)i;
            a = s[0];
            c = s[1];
            if (INAFF && !which) {
                a = bn_relu4(a, ldg4(p.in_scale + 8 * c8), ldg4(p.in_shift + 8 * c8));
                c = bn_relu4(c, ldg4(p.in_scale + 8 * c8 + 4), ldg4(p.in_shift + 8 * c8 + 4));
            }
            hi = reinterpret_cast<uint4 *>(o.dst + kHalfZeros) + (size_t)pix * (o.div8.d * 2) + (c8 >> 2) * 8 + (c8 & 3);
            mark = o.marks + (pix >> kHalfMarkShift);
        } else {
            // filters: (stage, chunk of eight, row), rows fastest where they lie next to each other in memory
            unsigned row, t;
            if (o.kind == kHalfFilter) {
                row = fdiv(i, o.div8);
                t = i - row * o.div8.d;  // eight elements of the row
            } else {
                t = fdiv(i, o.div8);     // div8.d: plane_rows
                row = i - t * o.div8.d;
            }
            const unsigned tap = fdiv(t * 8, o.div_k), kc = ((t * 8 - tap * o.div_k.d) >> 5) * o.taps + tap, q = t & 3;
            if ((int)row < o.rows) {
                if (o.kind == kHalfFilter) {
                    const float4 *s = reinterpret_cast<const float4 *>(o.src + (size_t)row * o.kdim) + 2 * t;
                    a = s[0];
                    c = s[1];
                } else {
                    // element (tap', k) of row c is w[k][taps - 1 - tap'][c]
                    const unsigned kk = t * 8, tapf = fdiv(kk, o.div_k), k0 = kk - tapf * o.div_k.d;
                    const float *s = o.src + ((size_t)k0 * o.taps + (o.taps - 1 - tapf)) * o.rows + row;
                    const size_t step = (size_t)o.taps * o.rows;
                    a = make_float4(s[0], s[step], s[2 * step], s[3 * step]);
                    c = make_float4(s[4 * step], s[5 * step], s[6 * step], s[7 * step]);
                }
            }
            const int sw = (row >> 1) & 7;
            uint4 *r = reinterpret_cast<uint4 *>(o.dst) + ((size_t)kc * o.plane_rows + row) * 8;
            hi = r + (q ^ sw);
            low_at = (int)((q + 4) ^ sw) - (int)(q ^ sw);
            mark = o.marks + row;
        }
        const float4 a0 = a, c0 = c;
        a = ldexp4(a, up);
        c = ldexp4(c, up);
        const Half8 h = half8(a, c);
        hi[0] = h.hi;
        hi[low_at] = h.lo;
        const unsigned tiny = tiny4(a0, a) + tiny4(c0, c);
        if (tiny) {
            atomicAdd(mark, tiny);
            *o.any = 1u;
        }
    }
}

// ---- implicit GEMM -----------------------------------------------------------------------------------------------------
// A wavefront's block as the kernels of this file hold it: blocks of 16 pixels x 16 channels, lane l has pixel l % 16 and channels 4 * (l / 16) .. + 3.
// Statistics (see igemm_stats: whole tiles only) and write-out, 16 bytes per lane.
template <int BM, int BN, bool STATS, int MI, int NI>
__device__ __forceinline__ void half_finish(const IgemmP &p, int lane, int wm, int wn, floatx4 (&acc)[MI][NI], float *part, int m0, int n0, int tm, float *s_mean,
                                            float *s_m2)
{
    constexpr int WTM = BM / 2, WTN = NI * 16;
    const int pl = lane & 15, cl = 4 * (lane >> 4);
    if (STATS && !part) {
        const int valid = min(WTM, p.M - (m0 + wm * WTM));  // rows of this wavefront inside the matrix (may be <= 0)
        const float cnt = valid > 0 ? 1.f / (float)valid : 0.f;
        float cmean[NI][4], cm2[NI][4];
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float sum = 0.f;
#pragma unroll
                for (int i = 0; i < MI; ++i) sum += i * 16 + pl < valid ? acc[i][j][e] : 0.f;
                const float mean = row16_sum(sum) * cnt;
                float dev = 0.f;
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const float d = acc[i][j][e] - mean;
                    dev = i * 16 + pl < valid ? fmaf(d, d, dev) : dev;
                }
                cmean[j][e] = mean;
                cm2[j][e] = row16_sum(dev);
                if (wm == 1 && pl == 0) {
                    s_mean[wn * WTN + j * 16 + cl + e] = cmean[j][e];
                    s_m2[wn * WTN + j * 16 + cl + e] = cm2[j][e];
                }
            }
        __syncthreads();  // the next write of s_mean comes after the barriers of the next item's loop
        if (wm == 0 && pl == 0) {
            const float na = (float)valid, nb = (float)max(0, min(WTM, p.M - (m0 + WTM)));
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int c = wn * WTN + j * 16 + cl, col = n0 + c;
                float4 mean, m2;
                float *mv = &mean.x, *dv = &m2.x;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    mv[e] = cmean[j][e];
                    dv[e] = cm2[j][e];
                    if (nb > 0.f) {
                        const float nt = na + nb, d = s_mean[c + e] - mv[e];
                        mv[e] = fmaf(d, nb / nt, mv[e]);
                        dv[e] = dv[e] + s_m2[c + e] + d * d * (na * nb / nt);
                    }
                }
                if (col < p.Nout) {
                    *reinterpret_cast<float4 *>(&p.stat_mean[(long)tm * p.Nout + col]) = mean;
                    *reinterpret_cast<float4 *>(&p.stat_m2[(long)tm * p.Nout + col]) = m2;
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int rl = wm * WTM + i * 16 + pl, m = m0 + rl;
        if (part) {
#pragma unroll
            for (int j = 0; j < NI; ++j) *reinterpret_cast<floatx4 *>(&part[rl * BN + wn * WTN + j * 16 + cl]) = acc[i][j];
        } else if (m < p.M) {
            const long row = out_row_index(p, m);
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int col = n0 + wn * WTN + j * 16 + cl;
                if (col >= p.Nout) continue;  // Nout % 4 == 0: the four columns are inside together
                *reinterpret_cast<floatx4 *>(&p.out[row * p.Nout + col]) = acc[i][j];
                if (p.scatter2 == 1) {
                    const floatx4 z = {0.f, 0.f, 0.f, 0.f};
                    *reinterpret_cast<floatx4 *>(&p.out[(row + 1) * p.Nout + col]) = z;
                    *reinterpret_cast<floatx4 *>(&p.out[(row + 2 * p.OW) * p.Nout + col]) = z;
                    *reinterpret_cast<floatx4 *>(&p.out[(row + 2 * p.OW + 1) * p.Nout + col]) = z;
                }
            }
        }
    }
}

// A wavefront's block formed on the fp32 instruction straight from memory (see igemm_join_split): results that are not finite, or
// operands that the halves do not hold.
constexpr int kAgainLoads = 2;  // groups of four elements: more take no less time, and registers that spill (16-byte loads: 1.4 - 1.9 times the time)
template <int MI, int NI>
__device__ __forceinline__ void half_again(const IgemmWideP &p, int lane, int mw, int nw, int first, int end, floatx4 (&acc)[MI][NI])
{
    const int pl = lane & 15, kl = lane >> 4;
    int ih0[MI], iw0[MI], base[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int m = mw + i * 16 + pl;
        int cls, n, oh, ow;
        decode_row(p, min(m, p.M - 1), cls, n, oh, ow);
        ih0[i] = m < p.M ? oh * p.so + p.off : -(1 << 28);
        iw0[i] = ow * p.so + p.off;
        base[i] = n * (p.IH * p.IW * p.Cin);
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    floatx4 run[MI][NI];  // sums of 128 elements, added up in acc
    for (int kc = first; kc < end; ++kc) {
        if ((kc - first) % kHalfFlush == 0)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    if (kc > first) acc[i][j] += run[i][j];
                    run[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
        const int chunk = (int)fdiv(kc, p.div_rs), tap = kc - chunk * (p.R * p.S);
        const int r = (int)fdiv(tap, p.div_s), sx = tap - r * p.S;
#pragma unroll 1
        for (int k2 = 0; k2 < kBK; k2 += 4 * kAgainLoads) {
            float va[kAgainLoads][MI], vb[kAgainLoads][NI];  // in flight together
#pragma unroll
            for (int q = 0; q < kAgainLoads; ++q) {
                const int c = chunk * kBK + k2 + 4 * q + kl;
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const int ih = ih0[i] + r, iw = iw0[i] + sx;
                    const bool ok = (unsigned)ih < (unsigned)p.IH && (unsigned)iw < (unsigned)p.IW;
                    va[q][i] = ok ? p.a[(unsigned)(base[i] + (ih * p.IW + iw) * p.Cin + c)] : 0.f;
                    if (p.in_scale && ok) va[q][i] = fmaxf(fmaf(va[q][i], p.in_scale[c], p.in_shift[c]), 0.f);
                }
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const int col = nw + j * 16 + pl;
                    vb[q][j] = 0.f;
                    if (col < p.Nout) {
                        if (p.flip_taps) {  // the filter as it is, [k][tap][row]: see half_split_kernel
                            vb[q][j] = p.b[((long)c * p.flip_taps + (p.flip_taps - 1 - tap)) * p.Nout + col];
                        } else {
                            vb[q][j] = p.b[(long)col * p.Kdim + tap * p.Cin + c];
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < kAgainLoads; ++q)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j) run[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vb[q][j], va[q][i], run[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] += run[i][j];
}

// The launch parameters read again where they are needed: held in scalar registers through the loop they spill into vector registers, and
// every stage then moves dozens of them.
__device__ __forceinline__ const IgemmWideP &again_from_memory()
{
    const char __attribute__((address_space(4))) *q = (const char __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(q));
    return *reinterpret_cast<const IgemmWideP *>((const char *)q);
}

// The implicit GEMM of igemm_kernel (its work decomposition; no dilation, Cin % 32 == 0, Nout % 4 == 0, R*S <= 32) on halves: a stage is 32 reduction elements, 64
// bytes of hi and 64 of lo in a row of the LDS image, and stages go through the filter taps of one group of 32 channels before the next group.
// What a stage costs beside its products is instructions (a wavefront issues one in four cycles, a product takes 16) and LDS reads (six fragments of
// 1 KB to 12 products with 64 x 32 to a wavefront, 128 bytes a cycle).  Three workgroups to a CU, each at another place of its stage, keep the
// matrix cores and the LDS busy at the same time; one of 128 x 128 with four stages in LDS had its wavefronts read and multiply in step.  3x3 256 -> 256,
// 14x14, N = 128 (29.6 GFLOP): 99 us in calls one behind the other, igemm_pre_kernel 179; that way 1.65 times as long, with addresses as igemm_act_kernel
// forms them 1.2 times.
template <int BM, int BN, bool STATS>
__global__ __launch_bounds__(kConvThreads, half_occupancy(BM, BN)) void igemm_half_kernel(IgemmWideP kernarg)
{
    constexpr int WTM = BM / 2, WTN = BN / 2, MI = WTM / 16, NI = WTN / 16;
    constexpr int RA = BM / 32, RB = BN / 32, STEP = 32;   // rows per thread: 8 threads copy a row
    constexpr int STAGE = (BM + BN) * 8;                   // 16-byte pieces
    __shared__ __attribute__((aligned(16))) uint4 S[2][STAGE];  // rows of the gathered tile, then the filter's
    __shared__ float s_stat[2][STATS ? BN : 1];
    main_chain_priority();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int G = gridDim.x, n_items = kernarg.full_items + kernarg.tail_tiles * kernarg.tail_split;
    int item = blockIdx.x;
    if (item >= n_items) return;

    // This thread copies LDS position tid%8 of rows tid/8 + 32*i, which holds chunk tid%8 ^ (tid/16 % 8) of each of them: of a row three
    // instructions, an addition of the stage's offset, the bit of the filter tap from a mask made once per item, and the choice of the zeros
    // ahead of the tensor.
    unsigned aoff[RA], amask[RA];
    auto set_rows = [&](const IgemmP &p, const IgemmItem &it) {
        const int t = opaque_tid(), arow = t >> 3;
        const unsigned ac = (unsigned)(((t & 7) ^ ((t >> 4) & 7)) * 16) + kHalfZeros;
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            const int m = it.m0 + arow + STEP * i;
            aoff[i] = amask[i] = 0;
            if (m < p.M) {
                int cls, n, oh, ow;
                decode_row(p, m, cls, n, oh, ow);
                const int ih = oh * p.so + p.off, iw = ow * p.so + p.off;
                unsigned bit = 1;
                for (int r = 0; r < p.R; ++r)
                    for (int s = 0; s < p.S; ++s, bit <<= 1) {
                        if ((unsigned)(ih + r) < (unsigned)p.IH && (unsigned)(iw + s) < (unsigned)p.IW) amask[i] |= bit;
                    }
                aoff[i] = (unsigned)((n * p.IH + ih) * p.IW + iw) * (unsigned)(p.Cin * 4) + ac;  // modulo 2^32, like the sums below
            }
        }
    };
    // The stage that is loaded next: chunk l_kc of an item, its tap, the offset of its tap and channels in the gathered tensor, its filter rows.
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_offset(&S[0][0]) + wave * 1024);
    const char *halves = kernarg.halves, *l_b;
    const unsigned px = kernarg.Cin * 4, row_jump = (kernarg.IW - kernarg.S) * px;
    const int taps = kernarg.R * kernarg.S, S_ = kernarg.S;
    const size_t b_step = (size_t)kernarg.plane_rows * kActRow;
    int l_kc, l_tap, l_s, buf = 0;
    unsigned l_delta, l_chunk;
    auto place = [&](const IgemmWideP &p, int kc, int n0) {
        l_kc = __builtin_amdgcn_readfirstlane(kc);
        const int chunk = __builtin_amdgcn_readfirstlane((int)fdiv(l_kc, p.div_rs));
        l_tap = l_kc - chunk * taps;
        const int r = __builtin_amdgcn_readfirstlane((int)fdiv(l_tap, p.div_s));
        l_s = l_tap - r * p.S;
        l_chunk = (unsigned)chunk * 128u;
        l_delta = (unsigned)(r * p.IW + l_s) * px + l_chunk;
        l_b = p.planes + ((size_t)l_kc * p.plane_rows + __builtin_amdgcn_readfirstlane(n0)) * kActRow;
    };
    auto start = [&](const IgemmWideP &p, const IgemmItem &x) {
        set_rows(p, x);
        place(p, x.kc_begin, x.n0);
    };
    auto load = [&]() {
        const unsigned lds = lds0 + buf * (STAGE * 16);
#pragma unroll
        for (int u = 0; u < RB; ++u) lds_copy16(l_b + u * 4096, tid * 16, lds + BM * kActRow + u * 4096);
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            const unsigned in = (unsigned)((int)(amask[i] << (31 - l_tap)) >> 31);  // the tap's bit in every bit
            lds_copy16(halves, (aoff[i] + l_delta) & in, lds + i * 4096);  // outside: the zeros ahead of the tensor
        }
    };
    // to the next stage of the item; false: there is none
    auto advance = [&](const IgemmItem &x) {
        if (++l_kc >= x.kc_end) return false;
        l_b += b_step;
        l_delta += px;
        if (++l_s == S_) {
            l_s = 0;
            l_delta += row_jump;
        }
        if (++l_tap == taps) {
            l_tap = l_s = 0;
            l_chunk += 128u;
            l_delta = l_chunk;
        }
        return true;
    };

    const int fa = act_chunk(wm * WTM + (lane & 15), lane >> 4), fb = BM * 8 + act_chunk(wn * WTN + (lane & 15), lane >> 4);
    const int lo_at = act_chunk(lane & 15, (lane >> 4) + 4) - act_chunk(lane & 15, lane >> 4);  // blocks of 16 rows share the swizzle
    floatx4 acc[MI][NI], top[MI][NI], low[MI][NI];  // finished sums of hi*hi, the running one, the small products'
    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
    auto multiply = [&]() {
        __builtin_amdgcn_s_setprio(3);
        const uint4 *q = S[buf];
        f16x8 bh[NI], bl[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            bl[j] = __builtin_bit_cast(f16x8, q[fb + j * 128 + lo_at]);
            bh[j] = __builtin_bit_cast(f16x8, q[fb + j * 128]);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const f16x8 ah = __builtin_bit_cast(f16x8, q[fa + i * 128]), al = __builtin_bit_cast(f16x8, q[fa + i * 128 + lo_at]);
#pragma unroll
            for (int j = 0; j < NI; ++j) low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bl[j], ah, low[i][j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NI; ++j) top[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bh[j], ah, top[i][j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NI; ++j) low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bh[j], al, low[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(2);
    };
    IgemmItem it = igemm_item<BM, BN>(kernarg, item, G);
    start(kernarg, it);
    load();
    bool drained = false;  // this stage's copies have been waited for already
    while (true) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = top[i][j] = low[i][j] = zero4;
        int run = 0;
        while (true) {
            if (!drained) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            drained = false;
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            const bool on = advance(it);
            if (!on) break;
            buf ^= 1;
            load();  // in flight while this stage is multiplied
            buf ^= 1;
            multiply();
            buf ^= 1;
            if (++run == kHalfFlush) {
                run = 0;
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            // the rest of the sum goes with the small products (exact where the larger number comes first)
                            const float t = top[i][j][e], s = acc[i][j][e] + t;
                            low[i][j][e] = fmaf(t - (s - acc[i][j][e]), (float)(1 << kHalfLow), low[i][j][e]);
                            acc[i][j][e] = s;
                        }
                        top[i][j] = zero4;
                    }
            }
        }
        // the item's last stage, with the first one of the next item on its way
        const IgemmWideP &p = again_from_memory();
        item += G;
        const bool more = item < n_items;
        IgemmItem nx = it;
        if (more) {
            nx = igemm_item<BM, BN>(p, item, G);
            start(p, nx);
            buf ^= 1;
            load();
            buf ^= 1;
        }
        multiply();
        buf ^= 1;
        const int down = -(p.half_up[0] + p.half_up[1]);
        const bool counted = __builtin_amdgcn_readfirstlane(p.half_any[0]) != 0;
        float probe = 0.f;  // NaN when a sum is not finite
        float sums[MI][NI];  // the least, over four outputs, of the largest magnitude of an output's three sums, which rarely cancel together
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                float m = 3.4e38f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float s = acc[i][j][e], t = top[i][j][e], l = low[i][j][e];
                    m = fminf(m, fmaxf(fmaxf(fabsf(s), fabsf(t)), 0.125f * fabsf(l)));
                    acc[i][j][e] = ldexpf(fmaf(l, 1.f / (float)(1 << kHalfLow), s + t), down);
                    probe = fmaf(acc[i][j][e], 0.f, probe);
                }
                // Now: put off to the branch that reads it, it would keep three sets of sums in registers, and those did not fit.  A launch of
                // 64 x 128 tiles with 36 bytes of scratch took 48.5 us, without 36.2 (3x3 128 -> 128, 28x28, N = 32, with statistics).
                asm volatile("" : "+v"(m));
                sums[i][j] = m;
            }
        bool again = probe != probe;
        const int l2 = opaque_tid() & 63;
        // A counted number loses at most 2^-20.4 of its scaled product (2^-37 of quantum and 2^-36 of the dropped lo*lo, times a number below 2^15).
        // An output one of whose sums shows that its products' magnitudes add up to 16 for each of them loses less than 2^-24 of that.
        // (|lo| is at most twice |hi|: its sums show it from 8 times as much on.)
        float least = 3.4e38f;
        if (counted) {
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const bool row = it.m0 + wm * WTM + i * 16 + (l2 & 15) < p.M;
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    if (row && it.n0 + wn * WTN + j * 16 + 4 * (l2 >> 4) < p.Nout) least = fminf(least, sums[i][j]);
                }
            }
        }
        const float elements = (float)((it.kc_end - it.kc_begin) * kBK);
        if (counted && __any(least < kHalfFloor * elements)) {  // their number under this block's rows (whole image rows), and in its filter rows
            const int mw = it.m0 + wm * WTM, nw = it.n0 + wn * WTN;
            int cls, n, oh, ow, n2, oh2, c2;
            decode_row(p, min(mw, p.M - 1), cls, n, oh, ow);
            decode_row(p, min(mw + WTM, p.M) - 1, c2, n2, oh2, ow);
            const int h0 = max(0, oh * p.so + p.off), h1 = min(p.IH - 1, oh2 * p.so + p.off + p.R - 1);
            const int g0 = ((n * p.IH + h0) * p.IW) >> kHalfMarkShift, g1 = ((n2 * p.IH + h1) * p.IW + p.IW - 1) >> kHalfMarkShift;
            float count = 0.f;
            for (int g = g0 + l2; g <= g1; g += 64) count += (float)p.half_marks[0][g];
            for (int g = nw + l2; g < min(nw + WTN, p.Nout); g += 64) count += (float)p.half_marks[1][g];
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) count += __shfl_xor(count, d, 64);
            again |= least < kHalfFloor * fminf(count, elements);  // none: never
        }
        if (__any(again))
            half_again(p, l2, it.m0 + wm * WTM, it.n0 + wn * WTN, it.kc_begin, it.kc_end, acc);
        drained = more;
        if (more) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the copies: from here on what is in flight are results
        half_finish<BM, BN, STATS>(p, l2, wm, wn, acc, it.part, it.m0, it.n0, it.tm, s_stat[0], s_stat[1]);
        if (!more) break;
        it = nx;
    }
}

}  // namespace rn50
