// Filter gradient with operands split into bf16 terms beforehand (device code; included by conv_terms.hip).  See split8 in conv_kernels.h for
// the products and their precision, which are wgrad_split_kernel's.
//
// What bounded that kernel (142 TFLOP/s on 3x3 256 -> 256, 14x14, N = 128) is the vector work of splitting: an element of dy is split once per tile of
// filter indices (18 times here), one of x once per tile of output channels and filter tap.  Here both tensors are split by one launch, 10 bytes
// of memory traffic per element, and copied to LDS without registers.  Products on v_mfma_f32_16x16x32_bf16: the same bits as on
// v_mfma_f32_32x32x16_bf16 at 12 % more of them within the chip's power (a loop of nothing else, operands of random bits).
#pragma once
#include "conv_act.h"

namespace rn50 {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// [pixel][C] fp32 (C % 32 == 0) -> [pixel][C/32][hi, mid, lo of 32 channels], 192 bytes to a group
template <bool INAFF>
static __global__ __launch_bounds__(256) void terms_prep_kernel(TermsPrep p)
{
    const int which = (int)blockIdx.x >= p.blocks[0], b = (int)blockIdx.x - (which ? p.blocks[0] : 0), tid = threadIdx.x;
    const unsigned n8 = p.n8[which], step = (unsigned)p.blocks[which] * 256u;
    const FastDiv div = p.div8[which];
    const float4 *src = reinterpret_cast<const float4 *>(p.src[which]);
    uint4 *dst = reinterpret_cast<uint4 *>(p.dst[which]);
    if (b == 0 && tid < kTermsZeros / 16) dst[tid] = make_uint4(0u, 0u, 0u, 0u);
    dst += kTermsZeros / 16;
    const float up = split_up();
    for (unsigned i = (unsigned)b * 256u + tid; i < n8; i += step) {
        const unsigned pix = fdiv(i, div), c8 = i - pix * div.d;
        float4 u = src[2 * (size_t)i], v = src[2 * (size_t)i + 1];
        if (INAFF && !which) {
            u = bn_relu4(u, ldg4(p.in_scale + 8 * c8), ldg4(p.in_shift + 8 * c8));
            v = bn_relu4(v, ldg4(p.in_scale + 8 * c8 + 4), ldg4(p.in_shift + 8 * c8 + 4));
        }
        const Split8 s = split8_scaled(scaled4(u, up), scaled4(v, up));
        uint4 *o = dst + (size_t)(i >> 2) * 12 + (i & 3);  // C % 32 == 0: groups of four follow each other across pixels
        o[0] = s.hi;
        o[4] = s.mid;
        o[8] = s.lo;
    }
}

// Eight bf16 of element order; a fragment's split elements keep the order of split8 (0-3, 16-19, ...): see the reads below.
// dw[k][j] = sum over pixels of dy[pixel][k] * xcol[pixel][j]: tiles, ranges and write-out of wgrad_split_kernel, copies of wgrad_act_copy_kernel.  LDS:
// [buffer][term][pixel row][channel]; 16-byte chunk c of row r at c ^ swz(r) (wgrad_act_swz).
template <int BM, int BN>
__global__ __launch_bounds__(kConvThreads, wgrad_terms_occupancy(BM, BN)) void wgrad_terms_kernel(WgradP p)
{
    constexpr int MI = BM / 32, NI = BN / 32;                      // blocks of 16 of a wavefront
    constexpr int CA = BM / 8, CB = BN / 8;                        // chunks per pixel row
    constexpr int RA = BM / 64, RB = BN / 64;                      // passes of the workgroup per term: 32 or 16 rows each
    constexpr int PA = kBK / RA, PB = kBK / RB;
    __shared__ __attribute__((aligned(16))) uint16_t As[2][3 * kBK * BM];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][3 * kBK * BN];

    const int ntiles = p.tiles_k * p.tiles_j;
    const int item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int split = item / ntiles, tile = item - split * ntiles;
    const int tk = tile / p.tiles_j, tj = tile - tk * p.tiles_j;
    const int k0 = tk * BM, j0 = tj * BN;
    const int pix_begin = split * p.pix_per_split, pix_end = min(p.Mpix, pix_begin + p.pix_per_split);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // this thread copies LDS position tid % CA (CB) of rows tid / CA + PA * i of every term; rows PA apart share the swizzle
    const int pa = tid / CA, pb = tid / CB;
    const int qa = (tid % CA) ^ wgrad_act_swz<BM>(pa), qb = (tid % CB) ^ wgrad_act_swz<BN>(pb);
    const bool kok = k0 + (qa >> 2) * 32 < p.Kout;  // Kout % 32 == 0
    const int j = j0 + (qb >> 2) * 32;              // Cin % 32 == 0: 32 indices share a filter tap
    const int r = j / (p.S * p.Cin), rem0 = j - r * (p.S * p.Cin), sx = rem0 / p.Cin, c = rem0 - sx * p.Cin;
    const int th = j < p.Jdim ? r - p.pad : -(1 << 28), tw = sx - p.pad;
    // byte offsets: 6 per element
    const unsigned toff = (unsigned)(((r - p.pad) * p.IW + tw) * p.Cin + c) * 6u + (unsigned)(qb & 3) * 16u + kTermsZeros;
    int apix = pix_begin + pa, bpix = pix_begin + pb, bih[RB], biw[RB];
    unsigned aoff = ((unsigned)apix * (unsigned)p.Kout + (unsigned)k0) * 6u + (unsigned)(qa >> 2) * 192u + (unsigned)(qa & 3) * 16u + kTermsZeros, boff[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int pix = bpix + PB * i;
        const int n = (int)fdiv(pix, p.div_ohw), rem = pix - n * (p.OH * p.OW);
        const int oh = (int)fdiv(rem, p.div_ow), ow = rem - oh * p.OW;
        bih[i] = oh * p.stride;
        biw[i] = ow * p.stride;
        boff[i] = ((unsigned)(n * p.IH + bih[i]) * (unsigned)p.IW + (unsigned)biw[i]) * (unsigned)p.Cin;
    }
    const unsigned astep = (unsigned)PA * (unsigned)p.Kout * 6u;
    const unsigned a_lds = lds_offset(&As[0][0]) + wave * 1024, b_lds = lds_offset(&Bs[0][0]) + wave * 1024;
    // copies the stage the running state points at, then advances the state by 32 pixels (see wgrad_fill); what does not exist: the zeros
    // ahead of the tensors
    auto load = [&](int buf) {
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            const bool ok = kok & (apix + PA * i < pix_end);
            const unsigned off = ok ? aoff + astep * i : 0u, term = ok ? 64u : 0u;
#pragma unroll
            for (int t = 0; t < 3; ++t) lds_copy16(p.dy_terms, off + term * t, a_lds + buf * (6 * kBK * BM) + (t * RA + i) * 4096);
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int ih = bih[i] + th, iw = biw[i] + tw;
            const bool ok = (bpix + PB * i < pix_end) & ((unsigned)ih < (unsigned)p.IH) & ((unsigned)iw < (unsigned)p.IW);
            const unsigned off = ok ? boff[i] * 6u + toff : 0u, term = ok ? 64u : 0u;
#pragma unroll
            for (int t = 0; t < 3; ++t) lds_copy16(p.x_terms, off + term * t, b_lds + buf * (6 * kBK * BN) + (t * RB + i) * 4096);
            biw[i] += p.adv_iw;
            boff[i] += p.adv_off;
            if (biw[i] >= p.lim_iw) {
                biw[i] -= p.lim_iw;
                bih[i] += p.stride;
                boff[i] += p.carry_row;
            }
            bih[i] += p.adv_ih;
            if (bih[i] >= p.lim_ih) {
                bih[i] -= p.lim_ih;
                boff[i] += p.carry_img;
            }
        }
        apix += kBK;
        bpix += kBK;
        aoff += p.adv_dy * 6u;
    };

    floatx4 acc[MI][NI], accl[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int n = 0; n < NI; ++n) acc[i][n] = accl[i][n] = floatx4{0.f, 0.f, 0.f, 0.f};
    // lane l reads four indices of pixel row frow (and of frow + 4: the same swizzle) and receives four pixels of index l % 16
    const int frow = 8 * (lane >> 4) + ((lane & 15) >> 2), fcol = (lane & 3) * 4;
    int ca[MI], cb[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int col = wm * (BM / 2) + i * 16 + fcol;
        ca[i] = frow * BM + (((col >> 3) ^ wgrad_act_swz<BM>(frow)) << 3) + (col & 7);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = wn * (BN / 2) + i * 16 + fcol;
        cb[i] = frow * BN + (((col >> 3) ^ wgrad_act_swz<BN>(frow)) << 3) + (col & 7);
    }
    auto frag = [&](const uint16_t *q, int pitch) {
        // rows frow + 4 have another swizzle where it follows more than the lowest two bits of the row: not here
        const Frag8 f = {lds_read_tr(q), lds_read_tr(q + 4 * pitch)};
        return __builtin_bit_cast(bf16x8, f);
    };
    const int stages = (pix_end - pix_begin + kBK - 1) / kBK;
    load(0);
    for (int st = 0; st < stages; ++st) {
        const int buf = st & 1;
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // this stage is there, the one before it has been read
        if (st + 1 < stages) load(buf ^ 1);
        __builtin_amdgcn_s_setprio(1);  // as in wgrad_tile: multiplying goes before address arithmetic, both below the main chain
        bf16x8 bf[3][NI];
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int n = 0; n < NI; ++n) bf[t][n] = frag(&Bs[buf][t * (kBK * BN) + cb[n]], BN);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            bf16x8 af[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) af[t] = frag(&As[buf][t * (kBK * BM) + ca[i]], BM);
#pragma unroll
            for (int pr = 0; pr < 6; ++pr) {
                constexpr int ta[6] = {0, 0, 1, 1, 0, 2}, tb[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
                for (int n = 0; n < NI; ++n) {
                    floatx4 &d = pr == 0 ? acc[i][n] : accl[i][n];
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[tb[pr]][n], af[ta[pr]], d, 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_s_setprio(0);
    }

    // block (i, n): lane l has output channel l % 16 and filter indices 4 * (l / 16) .. + 3
    const int l2 = opaque_tid() & 63, pl = l2 & 15, cl = 4 * (l2 >> 4);
    float probe = 0.f;  // NaN when a sum is not finite
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int n = 0; n < NI; ++n)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[i][n][e] = (acc[i][n][e] + accl[i][n][e]) * kSplitDown;
                probe = fmaf(acc[i][n][e], 0.f, probe);
            }
    if (__any(probe != probe)) {  // see igemm_join_split
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int n = 0; n < NI; ++n) acc[i][n] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int pix = pix_begin + (l2 >> 4); pix < pix_end + (l2 >> 4); pix += 4) {
            const bool in = pix < pix_end;
            const int pq = in ? pix : pix_begin;
            const int n0 = (int)fdiv(pq, p.div_ohw), rem = pq - n0 * (p.OH * p.OW);
            const int oh = (int)fdiv(rem, p.div_ow), ow = rem - oh * p.OW;
            float va[MI], vb[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int k = k0 + wm * (BM / 2) + i * 16 + pl;
                va[i] = in && k < p.Kout ? p.dy[(size_t)pq * p.Kout + k] : 0.f;
            }
#pragma unroll
            for (int n = 0; n < NI; ++n) {
                const int jj = j0 + wn * (BN / 2) + n * 16 + pl;
                const int rr = jj / (p.S * p.Cin), m0 = jj - rr * (p.S * p.Cin), ss = m0 / p.Cin, cc = m0 - ss * p.Cin;
                const int ih = oh * p.stride + rr - p.pad, iw = ow * p.stride + ss - p.pad;
                const bool ok = in && jj < p.Jdim && (unsigned)ih < (unsigned)p.IH && (unsigned)iw < (unsigned)p.IW;
                vb[n] = ok ? p.x[(((size_t)n0 * p.IH + ih) * p.IW + iw) * p.Cin + cc] : 0.f;
                if (p.in_scale && ok) vb[n] = fmaxf(fmaf(vb[n], p.in_scale[cc], p.in_shift[cc]), 0.f);
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int n = 0; n < NI; ++n) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(vb[n], va[i], acc[i][n], 0, 0, 0);
        }
    }
    float *out = p.out + (long)split * p.split_stride;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int k = k0 + wm * (BM / 2) + i * 16 + pl;
        if (k >= p.Kout) continue;
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int col = j0 + wn * (BN / 2) + n * 16 + cl;
            if (col < p.Jdim) *reinterpret_cast<floatx4 *>(&out[(long)k * p.Jdim + col]) = acc[i][n];  // Jdim % 32 == 0
        }
    }
}

}  // namespace rn50
