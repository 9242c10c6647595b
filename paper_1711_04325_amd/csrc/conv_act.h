// Implicit-GEMM kernel for activations kept as bfloat16 in memory (device code; included by conv_split.hip).
//
// What bounded the general kernel here (igemm_kernel with ACT = 1): every operand element passed through registers on its way
// to LDS (the filter in fp32, rounded there, once per row tile), two barriers a stage, and never more than one stage in
// flight.  With 2-byte operands a stage has so few matrix cycles that this is most of its time.  Here both operands are
// copied from memory to LDS without registers: the input's channels are gathered 16 bytes per lane (a lane whose filter tap
// lies outside the image copies zeros), and the filter was rounded to bf16 beforehand, once per call or once per training step, in
// the order of the LDS image.
#pragma once
#include "conv_split.h"

namespace rn50 {

constexpr int kActBK = 64;              // reduction elements per stage: a row of 128 bytes, eight 16-byte chunks
constexpr int kActRow = kActBK * 2;     // its bytes
// LDS image: chunk c of row r sits at c ^ (r/2 % 8): the 16 rows that a quarter of a fragment read touches fall into different banks.
__device__ inline int act_chunk(int row, int c) { return row * 8 + (c ^ ((row >> 1) & 7)); }

__device__ const uint4 g_zero16 = {0u, 0u, 0u, 0u};  // what lanes outside the image copy

// w [rows][Kdim] fp32 -> bf16, [Kdim/64][plane_rows][128 bytes] in the order of the LDS image; rows from `rows` on are zeros
__device__ inline void round_rows(const SplitJob &job, const float *__restrict__ src, char *__restrict__ dst, long idx)
{
    const int chunks = job.kdim / kActBK;
    const int c = (int)(idx & 7);
    const long t = idx >> 3;
    const int kc = (int)(t % chunks), j = (int)(t / chunks);
    if (j >= job.plane_rows) return;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (j < job.rows) {
        const float *p = src + (long)j * job.kdim + kc * kActBK + 8 * c;
        a = ldg4(p);
        b = ldg4(p + 4);
    }
    reinterpret_cast<uint4 *>(dst + ((long)kc * job.plane_rows + j) * kActRow)[c ^ ((j >> 1) & 7)] =
        make_uint4(bf16_pack2(a.x, a.y), bf16_pack2(a.z, a.w), bf16_pack2(b.x, b.y), bf16_pack2(b.z, b.w));
}
static __global__ __launch_bounds__(256) void filter_round_kernel(SplitJob job, const float *__restrict__ w, char *__restrict__ planes)
{
    round_rows(job, w, planes, (long)blockIdx.x * 256 + threadIdx.x);
}
static __global__ __launch_bounds__(256) void filter_round_batched_kernel(const SplitJob *__restrict__ jobs, int njobs, const float *__restrict__ base,
                                                                   char *__restrict__ planes)
{
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].block_begin <= (int)blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const SplitJob job = jobs[__builtin_amdgcn_readfirstlane(lo)];
    round_rows(job, base + job.src_off, planes + job.dst_off, (long)((int)blockIdx.x - job.block_begin) * 256 + threadIdx.x);
}

// 16 bytes per lane from each lane's own address to LDS (see lds_copy16)
__device__ __forceinline__ void lds_gather16(const void *addr, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(addr), "s"(lds) : "memory", "m0");
}

// Write-out of a tile of bf16 outputs.  As the accumulators lie, a store instruction writes two bytes per lane, 64 neighbouring bytes of two
// rows; a wavefront passes its block through LDS instead (`stage`: its own WTM x WTN elements, free of other use) and stores 16
// bytes per lane, whole lines.  Outputs with a row length that is not a multiple of 16 bytes go the direct way.  The 64 -> 256 channel layer at
// 56x56, N = 256, 411 MB of output: data gradient of 256 -> 64 205 -> 125 us, forward with statistics 300 -> 194.
template <int BM, int BN, bool STATS, int MI, int NI>
__device__ __forceinline__ void igemm_finish_act(const IgemmP &p, floatx16 (&acc)[MI][NI], float *part, int m0, int n0, int tm, float *s_mean, float *s_m2,
                                                 uint16_t *stage)
{
    const int tid = opaque_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    if (part || (p.Nout & 7)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        igemm_finish<BM, BN, true, STATS>(p, tid, wave, acc, part, m0, n0, tm, s_mean, s_m2);
        return;
    }
    igemm_stats<BM, BN, true, STATS>(p, tid, wave, acc, part, m0, n0, tm, s_mean, s_m2);
    constexpr int WTM = BM / 2, WTN = BN / 2, LPR = WTN / 8, RPI = 64 / LPR;  // lanes per row of 16-byte pieces, rows per instruction
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            const int rl = i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const uint32_t w = bf16_pack2(acc[i][j][e], acc[i][j][e + 1]);
                stage[rl * WTN + j * 32 + (lane & 31)] = (uint16_t)w;
                stage[(rl + 1) * WTN + j * 32 + (lane & 31)] = (uint16_t)(w >> 16);
            }
        }
    // this wavefront's own stores to LDS (no other one touches them), and the copies of the next stage: from here on what is in flight
    // are results, which the next stage does not wait for
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    const int c8 = lane % LPR, col = n0 + wn * WTN + c8 * 8;
    bf16_t *out = reinterpret_cast<bf16_t *>(p.out);
#pragma unroll
    for (int q = 0; q < WTM / RPI; ++q) {
        const int rl = q * RPI + lane / LPR, m = m0 + wm * WTM + rl;
        const uint4 v = *reinterpret_cast<const uint4 *>(&stage[rl * WTN + c8 * 8]);
        if (m >= p.M || col >= p.Nout) continue;
        const long row = out_row_index(p, m);
        uint4 *o = reinterpret_cast<uint4 *>(out + row * p.Nout + col);
        *o = v;
        if (p.scatter2 == 1) {
            const uint4 z = make_uint4(0u, 0u, 0u, 0u);
            *reinterpret_cast<uint4 *>(out + (row + 1) * p.Nout + col) = z;
            *reinterpret_cast<uint4 *>(out + (row + 2 * p.OW) * p.Nout + col) = z;
            *reinterpret_cast<uint4 *>(out + (row + 2 * p.OW + 1) * p.Nout + col) = z;
        }
    }
}

// MODE 0: no dilation; 1: dilation 2 (strided data gradient).  Cin % 64 == 0.  Work decomposition, statistics and write-out are
// igemm_kernel's.  One barrier per stage: behind it this stage's copies have landed (each wavefront has waited for its own) and
// every wavefront has read the stage before, whose buffers then receive the next one.
template <int BM, int BN, int MODE, bool STATS>
__global__ __launch_bounds__(kConvThreads, igemm_act_occupancy(BM, BN)) void igemm_act_kernel(IgemmP p)
{
    constexpr int WTM = BM / 2, WTN = BN / 2, MI = WTM / 32, NI = WTN / 32;
    constexpr int RA = BM / 32, RB = BN / 32;   // rows per thread: 8 threads copy a row
    __shared__ __attribute__((aligned(16))) uint4 Bs[2][BN * 8];
    __shared__ __attribute__((aligned(16))) uint4 As[2][BM * 8];
    __shared__ float s_stat[2][STATS ? BN : 1];
    main_chain_priority();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int G = gridDim.x, n_items = p.full_items + p.tail_tiles * p.tail_split;
    int item = blockIdx.x;
    if (item >= n_items) return;
    const char *a8 = reinterpret_cast<const char *>(p.a);

    // this thread copies LDS position tid%8 of rows tid/8 + 32*i, which holds chunk tid%8 ^ (tid/16 % 8) of each of them
    const int arow = tid >> 3, ac = ((tid & 7) ^ ((tid >> 4) & 7)) * 8;
    int hn[RA], wnum[RA];
    unsigned abase[RA];
    int skip_ph = -1, skip_pw = 0;
    auto set_rows = [&](const IgemmItem &it) {
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            const int m = it.m0 + arow + 32 * i;
            hn[i] = -(1 << 28);
            wnum[i] = 0;
            abase[i] = 0;
            if (m < p.M) {
                int cls, n, oh, ow;
                decode_row(p, m, cls, n, oh, ow);
                if (p.scatter2 == 2) {
                    oh = 2 * oh + (cls >> 1);
                    ow = 2 * ow + (cls & 1);
                }
                hn[i] = oh * p.so + p.off;
                wnum[i] = ow * p.so + p.off;
                abase[i] = (unsigned)(n * (p.IH * p.IW * p.Cin) + ac);
            }
        }
        if (MODE == 1 && p.scatter2 == 2) {
            const int mq = p.M >> 2, c0 = it.m0 / mq, c1 = min(it.m0 + BM - 1, p.M - 1) / mq;
            skip_ph = c0 == c1 ? c0 >> 1 : -1;
            skip_pw = c0 & 1;
        }
    };
    auto next_chunk = [&](int kc, int end, int ph, int pw) {
        if (MODE != 1 || ph < 0) return kc;
        for (; kc < end; ++kc) {
            const int tap = (int)fdiv(kc * kActBK, p.div_cin);
            const int r = (int)fdiv(tap, p.div_s), sx = tap - r * p.S;
            if ((((ph + p.off + r) | (pw + p.off + sx)) & 1) == 0) break;
        }
        return kc;
    };
    auto first_chunk = [&](const IgemmItem &it) {
        const int kc = next_chunk(it.kc_begin, it.kc_end, skip_ph, skip_pw);
        return kc < it.kc_end ? kc : it.kc_begin;
    };
    const unsigned b_lds = lds_offset(&Bs[0][0]) + wave * 1024, a_lds = lds_offset(&As[0][0]) + wave * 1024;
    auto load = [&](int n0, int kc, int buf) {
        const char *src = p.planes + ((size_t)kc * p.plane_rows + n0) * kActRow;
#pragma unroll
        for (int u = 0; u < RB; ++u) lds_copy16(src + u * 4096, tid * 16, b_lds + buf * (BN * kActRow) + u * 4096);
        const int k0 = kc * kActBK;
        const int tap = (int)fdiv(k0, p.div_cin);
        const int c0 = k0 - tap * p.Cin;
        const int r = (int)fdiv(tap, p.div_s), s = tap - r * p.S;
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            int ih = hn[i] + r, iw = wnum[i] + s;
            bool ok = ih >= 0 && iw >= 0;
            if (MODE == 1) {
                ok = ok && ((ih | iw) & 1) == 0;
                ih >>= 1;
                iw >>= 1;
            }
            ok = ok && ih < p.IH && iw < p.IW;
            const unsigned aoff = abase[i] + (unsigned)((int)__umul24(__umul24(ih, p.IW) + iw, p.Cin) + c0);
            const char *q = ok ? a8 + (size_t)aoff * 2 : reinterpret_cast<const char *>(&g_zero16);
            lds_gather16(q, a_lds + buf * (BM * kActRow) + i * 4096);
        }
    };

    floatx16 acc[MI][NI];
    IgemmItem it = igemm_item<BM, BN>(p, item, G);
    set_rows(it);
    int kc = first_chunk(it), buf = 0;
    load(it.n0, kc, 0);
    auto compute = [&]() {
        __builtin_amdgcn_s_setprio(3);
        const uint4 *aq = As[buf], *bq = Bs[buf];
#pragma unroll
        for (int ks = 0; ks < kActBK / 16; ++ks) {
            const int c = ks * 2 + (lane >> 5);
            uint4 af[MI], bf[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) af[i] = aq[act_chunk(wm * WTM + i * 32 + (lane & 31), c)];
#pragma unroll
            for (int j = 0; j < NI; ++j) bf[j] = bq[act_chunk(wn * WTN + j * 32 + (lane & 31), c)];
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i]), __builtin_bit_cast(bf16x8, bf[j]), acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(2);
    };
    bool drained = false;  // this stage's copies have been waited for already
    while (true) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
        const int ph = skip_ph, pw = skip_pw;
        for (int kn; (kn = next_chunk(kc + 1, it.kc_end, ph, pw)) < it.kc_end; kc = kn) {
            if (!drained) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            drained = false;
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            load(it.n0, kn, buf ^ 1);  // in flight while this stage is multiplied
            compute();
            buf ^= 1;
        }
        // the item's last stage, with the first one of the next item on its way
        if (!drained) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        item += G;
        const bool more = item < n_items;
        IgemmItem nx = it;
        if (more) {
            nx = igemm_item<BM, BN>(p, item, G);
            set_rows(nx);
            kc = first_chunk(nx);
            load(nx.n0, kc, buf ^ 1);
        }
        compute();
        if (MODE == 1 && next_chunk(it.kc_begin, it.kc_end, ph, pw) >= it.kc_end) {
            // no stage reaches this item: it has multiplied one of zeros, of which an infinite weight makes NaNs
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
        }
        buf ^= 1;
        drained = true;  // igemm_finish_act waits for the copies before it stores
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // every wavefront has read the last stage: its buffers stage the write-out
        uint16_t *stage = reinterpret_cast<uint16_t *>(wave < 2 ? As[buf ^ 1] : Bs[buf ^ 1]) + (wave & 1) * (WTM * WTN);
        igemm_finish_act<BM, BN, STATS>(p, acc, it.part, it.m0, it.n0, it.tm, s_stat[0], s_stat[1], stage);
        if (!more) break;
        it = nx;
    }
}

// ---- filter gradient -------------------------------------------------------------------------------------------------
// dw[k][j] = sum over pixels of dy[pixel][k] * xcol[pixel][j], both tensors bf16: tiles of BM x BN, partial sums in fp32 over a pixel range,
// as wgrad_kernel.  wgrad_act_kernel (64 x 64 tiles, two products between barriers, operands transposed word by word on their way
// through registers) spent its time on the latency of its loads: 1.5 us per stage of 32 pixels.  Here stages of 64 pixels are
// copied to LDS as they lie in memory, [pixel][index], one stage ahead, and read back with the transposing LDS read.
// 16-byte chunk c of pixel row r sits at c ^ swz(r): the four rows of 32 indices that half a wavefront reads lie in 64 different banks.
template <int B>
__device__ __forceinline__ int wgrad_act_swz(int row) { return B == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }

// INAFF: x is max(0, x*in_scale[c] + in_shift[c]) rounded to bf16 (the BN + ReLU output as stored): it passes through registers on its
// way, in the same places, so the sums are those of the tensor as it would have been written.
template <int BM, int BN, bool INAFF>
__global__ __launch_bounds__(kConvThreads, igemm_act_occupancy(BM, BN)) void wgrad_act_copy_kernel(WgradP p)
{
    constexpr int MI = BM / 64, NI = BN / 64;
    constexpr int CA = BM / 8, CB = BN / 8;                        // chunks per pixel row
    constexpr int PA = kConvThreads / CA, PB = kConvThreads / CB;  // pixel rows per pass of the workgroup
    constexpr int RA = kActBK / PA, RB = kActBK / PB;
    __shared__ __attribute__((aligned(16))) uint16_t As[2][kActBK * BM];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][kActBK * BN];

    const int ntiles = p.tiles_k * p.tiles_j;
    const int item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int split = item / ntiles, tile = item - split * ntiles;
    const int tk = tile / p.tiles_j, tj = tile - tk * p.tiles_j;
    const int k0 = tk * BM, j0 = tj * BN;
    const int pix_begin = split * p.pix_per_split, pix_end = min(p.Mpix, pix_begin + p.pix_per_split);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // this thread copies LDS position tid % CA (CB) of rows tid / CA + PA * i: the swizzle is the same for all of them
    const int pa = tid / CA, pb = tid / CB;
    const int ka = k0 + ((tid % CA) ^ wgrad_act_swz<BM>(pa)) * 8, j = j0 + ((tid % CB) ^ wgrad_act_swz<BN>(pb)) * 8;
    const bool jok = j < p.Jdim, kok = ka < p.Kout;  // eight indices share a filter tap (Cin % 8 == 0) and end together (Kout % 8 == 0)
    const int r = j / (p.S * p.Cin), rem0 = j - r * (p.S * p.Cin), sx = rem0 / p.Cin, c = rem0 - sx * p.Cin;
    const int th = r - p.pad, tw = sx - p.pad, toff = (th * p.IW + tw) * p.Cin + c;
    int apix = pix_begin + pa, bpix = pix_begin + pb, bih[RB], biw[RB];
    unsigned aoff = (unsigned)apix * (unsigned)p.Kout + (unsigned)ka, boff[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int pix = bpix + PB * i;
        const int n = (int)fdiv(pix, p.div_ohw), rem = pix - n * (p.OH * p.OW);
        const int oh = (int)fdiv(rem, p.div_ow), ow = rem - oh * p.OW;
        bih[i] = oh * p.stride;
        biw[i] = ow * p.stride;
        boff[i] = ((unsigned)(n * p.IH + bih[i]) * (unsigned)p.IW + (unsigned)biw[i]) * (unsigned)p.Cin;
    }
    float4 in_sc[2] = {}, in_sh[2] = {};
    uint4 held[INAFF ? RB : 1];
    unsigned in_ok = 0;
    if (INAFF && jok) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            in_sc[t] = ldg4(p.in_scale + c + 4 * t);
            in_sh[t] = ldg4(p.in_shift + c + 4 * t);
        }
    }
    const char *dy8 = reinterpret_cast<const char *>(p.dy), *x8 = reinterpret_cast<const char *>(p.x), *zero = reinterpret_cast<const char *>(&g_zero16);
    const unsigned a_lds = lds_offset(&As[0][0]) + wave * 1024, b_lds = lds_offset(&Bs[0][0]) + wave * 1024;
    // copies the stage the running state points at, then advances the state by 64 pixels (two of wgrad_fill's advances of kBK)
    auto load = [&](int buf) {
        const unsigned astep = (unsigned)PA * (unsigned)p.Kout;
#pragma unroll
        for (int i = 0; i < RA; ++i)
            lds_gather16(kok && apix + PA * i < pix_end ? dy8 + (size_t)(aoff + astep * i) * 2 : zero, a_lds + buf * (kActBK * BM * 2) + i * 4096);
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int ih = bih[i] + th, iw = biw[i] + tw;
            const bool ok = (bpix + PB * i < pix_end) & jok & ((unsigned)ih < (unsigned)p.IH) & ((unsigned)iw < (unsigned)p.IW);
            const char *q = ok ? x8 + (size_t)(boff[i] + (unsigned)toff) * 2 : zero;
            if (INAFF) {
                held[i] = *reinterpret_cast<const uint4 *>(q);
                in_ok = i == 0 ? (unsigned)ok : in_ok | (unsigned)ok << i;
            } else {
                lds_gather16(q, b_lds + buf * (kActBK * BN * 2) + i * 4096);
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) {
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
        }
        apix += kActBK;
        bpix += kActBK;
        aoff += 2 * p.adv_dy;
    };

    auto put_held = [&](int buf) {  // INAFF: the rows load() left in registers
#pragma unroll
        for (int i = 0; i < (INAFF ? RB : 0); ++i) {
            uint4 v = held[i];
            if (in_ok & (1u << i)) {  // padding stays zero
                v.x = bf16_pack2(fmaxf(fmaf(bf16_lo(v.x), in_sc[0].x, in_sh[0].x), 0.f), fmaxf(fmaf(bf16_hi(v.x), in_sc[0].y, in_sh[0].y), 0.f));
                v.y = bf16_pack2(fmaxf(fmaf(bf16_lo(v.y), in_sc[0].z, in_sh[0].z), 0.f), fmaxf(fmaf(bf16_hi(v.y), in_sc[0].w, in_sh[0].w), 0.f));
                v.z = bf16_pack2(fmaxf(fmaf(bf16_lo(v.z), in_sc[1].x, in_sh[1].x), 0.f), fmaxf(fmaf(bf16_hi(v.z), in_sc[1].y, in_sh[1].y), 0.f));
                v.w = bf16_pack2(fmaxf(fmaf(bf16_lo(v.w), in_sc[1].z, in_sh[1].z), 0.f), fmaxf(fmaf(bf16_hi(v.w), in_sc[1].w, in_sh[1].w), 0.f));
            }
            reinterpret_cast<uint4 *>(Bs[buf])[tid + kConvThreads * i] = v;
        }
    };

    floatx16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int n = 0; n < NI; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][n][e] = 0.f;
    // lane l reads four indices of pixel row frow (+4, +16, ...: the same swizzle) and receives four pixels of index l % 16
    const int frow = 8 * (lane >> 5) + ((lane & 15) >> 2), fcol = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    int ca[MI], cb[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int col = wm * (BM / 2) + i * 32 + fcol;
        ca[i] = frow * BM + (((col >> 3) ^ wgrad_act_swz<BM>(frow)) << 3) + (col & 7);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = wn * (BN / 2) + i * 32 + fcol;
        cb[i] = frow * BN + (((col >> 3) ^ wgrad_act_swz<BN>(frow)) << 3) + (col & 7);
    }
    const int stages = (pix_end - pix_begin + kActBK - 1) / kActBK;
    load(0);
    if (INAFF) put_held(0);
    for (int st = 0; st < stages; ++st) {
        const int buf = st & 1;
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // this stage is there, the one before it has been read
        if (st + 1 < stages) load(buf ^ 1);
        __builtin_amdgcn_s_setprio(1);  // as in wgrad_tile: multiplying goes before address arithmetic, both below the main chain
#pragma unroll
        for (int ks = 0; ks < kActBK / 16; ++ks) {
            Frag8 af[MI], bf[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const uint16_t *q = &As[buf][ca[i] + ks * 16 * BM];
                af[i] = Frag8{lds_read_tr(q), lds_read_tr(q + 4 * BM)};
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const uint16_t *q = &Bs[buf][cb[i] + ks * 16 * BN];
                bf[i] = Frag8{lds_read_tr(q), lds_read_tr(q + 4 * BN)};
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int n = 0; n < NI; ++n)
                    acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i]), __builtin_bit_cast(bf16x8, bf[n]), acc[i][n], 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(0);
        if (INAFF && st + 1 < stages) put_held(buf ^ 1);  // those buffers were read one stage ago, before this stage's barrier
    }
    const int l2 = opaque_tid() & 63;
    float *out = p.out + (long)split * p.split_stride;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int k = k0 + wm * (BM / 2) + i * 32 + 8 * (e >> 2) + 4 * (l2 >> 5) + (e & 3);
            if (k >= p.Kout) continue;
#pragma unroll
            for (int n = 0; n < NI; ++n) {
                const int col = j0 + wn * (BN / 2) + n * 32 + (l2 & 31);
                if (col < p.Jdim) out[(long)k * p.Jdim + col] = acc[i][n][e];
            }
        }
}

}  // namespace rn50
