// fp32 implicit-GEMM kernels whose filter operand was split into its bf16 terms beforehand (device code; included by
// conv_split.hip).  See split8 in conv_kernels.h for the products and their precision.
//
// What bounds the general kernel (igemm_kernel) once its products run on the bf16 matrix instruction is the vector work of
// splitting: 6.5 instructions per operand element and stage, as many cycles as the matrix work of a 64-wide tile.  The
// filter is the same for every row tile, so here it is split once per call (or once per training step), stored in the
// order and bank swizzle of the LDS image, and copied from memory to LDS without passing through registers.
#pragma once
#include "conv_kernels.h"

namespace rn50 {

constexpr int kPlaneRow = kSplitRow * 4;  // bytes of one filter row's 32 split elements

// w [rows][Kdim] fp32 -> planes [Kdim/32][plane_rows][192 bytes]: stage kc of filter row j as split_chunk lays it out (the
// swizzle depends on j modulo 16 only, so a tile that starts at a multiple of 16 rows is copied to LDS as it is).  Rows from
// `rows` to plane_rows are zeros.  One thread per (stage, row, chunk of eight elements).
typedef SplitJobHost SplitJob;
__device__ inline void split_rows(const SplitJob &job, const float *__restrict__ src, char *__restrict__ dst, long idx)
{
    const int chunks = job.kdim / kBK;
    const int c = (int)(idx & 3);
    // consecutive threads: the chunks of one row's stages, so that a wavefront reads whole lines of the filter
    const long t = idx >> 2;
    const int kc = (int)(t % chunks), j = (int)(t / chunks);
    if (j >= job.plane_rows) return;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (j < job.rows) {
        const float *p = src + (long)j * job.kdim + kc * kBK + 4 * c;
        a = ldg4(p);
        b = ldg4(p + 16);
    }
    const Split8 v = split8(a, b, split_up());
    uint4 *o = reinterpret_cast<uint4 *>(dst + ((long)kc * job.plane_rows + j) * kPlaneRow) + (c ^ ((j >> 2) & 3));
    o[0] = v.hi;
    o[4] = v.mid;
    o[8] = v.lo;
}
static __global__ __launch_bounds__(256) void filter_split_kernel(SplitJob job, const float *__restrict__ w, char *__restrict__ planes)
{
    split_rows(job, w, planes, (long)blockIdx.x * 256 + threadIdx.x);
}
// All filters of a network in one launch: job j owns workgroups [block_begin, next job's block_begin).
static __global__ __launch_bounds__(256) void filter_split_batched_kernel(const SplitJob *__restrict__ jobs, int njobs, const float *__restrict__ base,
                                                                   char *__restrict__ planes)
{
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].block_begin <= (int)blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const SplitJob job = jobs[__builtin_amdgcn_readfirstlane(lo)];
    split_rows(job, base + job.src_off, planes + job.dst_off, (long)((int)blockIdx.x - job.block_begin) * 256 + threadIdx.x);
}

// 1024 bytes from memory to LDS, 16 per lane, without registers: lane l's bytes at gbase + voff go to lds + 16*l.  gbase and lds
// are the same for the whole wavefront.  The copy counts against vmcnt like a load; the compiler does not know of it, so the
// kernels wait for it themselves.
__device__ __forceinline__ void lds_copy16(const void *gbase, unsigned voff, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(gbase), "s"(lds) : "memory", "m0");
}
// Byte offset of a __shared__ object in the workgroup's LDS.
__device__ inline unsigned lds_offset(const void *p)
{
    return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}

struct IgemmItem {
    int m0, n0, tm, kc_begin, kc_end;
    float *part;
};
template <int BM, int BN>
__device__ __forceinline__ IgemmItem igemm_item(const IgemmP &p, int item, int G)
{
    IgemmItem it;
    int tile;
    it.part = nullptr;
    if (item < p.full_items) {  // see igemm_kernel: each XCD takes a contiguous range of the tiles of a round
        const int round = item / G, i = item - round * G;
        tile = round * G + (i & 7) * (G >> 3) + (i >> 3);
        it.kc_begin = 0;
        it.kc_end = p.kchunks;
    } else {
        const int piece = item - p.full_items;
        const int tt = piece / p.tail_split, sp = piece - tt * p.tail_split;
        tile = p.full_items + tt;
        it.kc_begin = sp * p.tail_chunks;
        it.kc_end = min(p.kchunks, it.kc_begin + p.tail_chunks);
        if (p.tail_split > 1) it.part = p.partial + (long)piece * (BM * BN);
    }
    it.tm = tile / p.tiles_n;
    it.m0 = it.tm * BM;
    it.n0 = (tile - it.tm * p.tiles_n) * BN;
    return it;
}

// One 16-element half of a stage: six products per pair of blocks, the hi*hi ones into acc, the others into accl.
// a_at(i), b_at(j): the 16-byte LDS words of this lane's hi fragment of row block i, column block j (mid and lo follow four words apart).
template <int MI, int NI, class AAt, class BAt>
__device__ __forceinline__ void split_products(const uint4 *aq, const uint4 *bq, AAt a_at, BAt b_at, floatx16 (&acc)[MI][NI], floatx16 (&accl)[MI][NI])
{
    uint4 af[MI][3], bf[NI][3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
#pragma unroll
        for (int i = 0; i < MI; ++i) af[i][t] = aq[a_at(i) + 4 * t];
#pragma unroll
        for (int j = 0; j < NI; ++j) bf[j][t] = bq[b_at(j) + 4 * t];
    }
#pragma unroll
    for (int pr = 0; pr < 6; ++pr) {
        constexpr int ta[6] = {0, 0, 1, 1, 0, 2}, tb[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                floatx16 &d = pr == 0 ? acc[i][j] : accl[i][j];
                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i][ta[pr]]), __builtin_bit_cast(bf16x8, bf[j][tb[pr]]), d, 0, 0, 0);
            }
    }
}
template <int MI, int NI>
__device__ __forceinline__ void clear_acc(floatx16 (&acc)[MI][NI], floatx16 (&accl)[MI][NI])
{
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = accl[i][j][e] = 0.f;
}

// The implicit GEMM of igemm_kernel (same work decomposition, MODE 0 and, for a dilation of 2, MODE 1; Cin % 32 == 0) with p.planes as filter operand.
// Stages follow each other across work items: the first stage of a workgroup's next item is loaded while the last stage of the
// present one is multiplied, and an item's results are stored behind the barrier wait of those loads.
template <int BM, int BN, int MODE, bool INAFF, bool STATS>
__global__ __launch_bounds__(kConvThreads, igemm_pre_occupancy(BM, BN)) void igemm_pre_kernel(IgemmP p)
{
    constexpr int WTM = BM / 2, WTN = BN / 2, MI = WTM / 32, NI = WTN / 32;
    constexpr int RA = BM / 64;            // rows of the gathered tile per thread, eight elements of each (4 threads per row)
    constexpr int NB = BN * 12 / kConvThreads;  // 16-byte pieces of a filter stage per thread
    __shared__ __attribute__((aligned(16))) uint4 Bs[2][BN * 12];
    __shared__ __attribute__((aligned(16))) uint4 As[BM * 12];
    __shared__ float s_stat[2][STATS ? BN : 1];
    main_chain_priority();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int q = tid & 3, arow = tid >> 2;
    const int G = gridDim.x, n_items = p.full_items + p.tail_tiles * p.tail_split;
    int item = blockIdx.x;
    if (item >= n_items) return;

    // geometry of this thread's rows of the item whose stages are being loaded (see igemm_kernel)
    int hn[RA], wnum[RA], abase[RA];
    int skip_ph = -1, skip_pw = 0;
    auto set_rows = [&](const IgemmItem &it) {
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            const int m = it.m0 + arow + 64 * i;
            hn[i] = -(1 << 28);
            wnum[i] = abase[i] = 0;
            if (m < p.M) {
                int cls, n, oh, ow;
                decode_row(p, m, cls, n, oh, ow);
                if (p.scatter2 == 2) {
                    oh = 2 * oh + (cls >> 1);
                    ow = 2 * ow + (cls & 1);
                }
                hn[i] = oh * p.so + p.off;
                wnum[i] = ow * p.so + p.off;
                abase[i] = n * (p.IH * p.IW * p.Cin);
            }
        }
        if (MODE == 1 && p.scatter2 == 2) {
            const int mq = p.M >> 2, c0 = it.m0 / mq, c1 = min(it.m0 + BM - 1, p.M - 1) / mq;
            skip_ph = c0 == c1 ? c0 >> 1 : -1;
            skip_pw = c0 & 1;
        }
    };
    // the next stage from kc on whose filter tap reaches a row of the tile
    auto next_chunk = [&](int kc, int end, int ph, int pw) {
        if (MODE != 1 || ph < 0) return kc;
        for (; kc < end; ++kc) {
            const int tap = (int)fdiv(kc * kBK, p.div_cin);
            const int r = (int)fdiv(tap, p.div_s), sx = tap - r * p.S;
            if ((((ph + p.off + r) | (pw + p.off + sx)) & 1) == 0) break;
        }
        return kc;
    };
    // an item none of whose stages reaches it multiplies one stage of zeros
    auto first_chunk = [&](const IgemmItem &it) {
        const int kc = next_chunk(it.kc_begin, it.kc_end, skip_ph, skip_pw);
        return kc < it.kc_end ? kc : it.kc_begin;
    };

    const unsigned b_lds = lds_offset(&Bs[0][0]) + wave * 1024;
    auto load_b = [&](int n0, int kc, int buf) {
        const char *src = p.planes + ((size_t)kc * p.plane_rows + n0) * kPlaneRow;
#pragma unroll
        for (int u = 0; u < NB; ++u) lds_copy16(src + u * 4096, tid * 16, b_lds + buf * (BN * kPlaneRow) + u * 4096);
    };
    float4 ra[RA][2];
    float4 in_sc[2], in_sh[2];
    unsigned in_ok = 0;
    auto load_a = [&](int kc) {
        const int k0 = kc * kBK;
        const int tap = (int)fdiv(k0, p.div_cin);
        const int c0 = k0 - tap * p.Cin + q * 4;
        const int r = (int)fdiv(tap, p.div_s), s = tap - r * p.S;
        if (INAFF) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                in_sc[t] = ldg4(p.in_scale + c0 + 16 * t);
                in_sh[t] = ldg4(p.in_shift + c0 + 16 * t);
            }
            in_ok = 0;
        }
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
            const unsigned aoff = (unsigned)(abase[i] + (int)__umul24(__umul24(ih, p.IW) + iw, p.Cin) + c0);
#pragma unroll
            for (int t = 0; t < 2; ++t) ra[i][t] = ok ? ldg4(p.a + (aoff + 16 * t)) : make_float4(0.f, 0.f, 0.f, 0.f);
            if (INAFF && ok) in_ok |= 1u << i;
        }
    };
    auto store_a = [&]() {
        const float up = split_up();
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            if (INAFF && (in_ok & (1u << i))) {
                ra[i][0] = bn_relu4(ra[i][0], in_sc[0], in_sh[0]);
                ra[i][1] = bn_relu4(ra[i][1], in_sc[1], in_sh[1]);
            }
            const Split8 v = split8(ra[i][0], ra[i][1], up);
            const int at = split_chunk(arow + 64 * i, 0, q);
            As[at] = v.hi;
            As[at + 4] = v.mid;
            As[at + 8] = v.lo;
        }
    };

    floatx16 acc[MI][NI], accl[MI][NI];
    IgemmItem it = igemm_item<BM, BN>(p, item, G);
    set_rows(it);
    int kc = first_chunk(it), buf = 0;
    load_b(it.n0, kc, 0);
    load_a(kc);
    store_a();
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    auto compute = [&]() {
        __builtin_amdgcn_s_setprio(3);
        const uint4 *bq = Bs[buf];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int c = ks * 2 + (lane >> 5);
            split_products<MI, NI>(As, bq, [&](int i) { return split_chunk(wm * WTM + i * 32 + (lane & 31), 0, c); },
                                   [&](int j) { return split_chunk(wn * WTN + j * 32 + (lane & 31), 0, c); }, acc, accl);
        }
        __builtin_amdgcn_s_setprio(2);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // every fragment of this stage has been read
    };
    while (true) {
        const int ph = skip_ph, pw = skip_pw;
        clear_acc(acc, accl);
        for (int kn; (kn = next_chunk(kc + 1, it.kc_end, ph, pw)) < it.kc_end; kc = kn) {
            load_b(it.n0, kn, buf ^ 1);  // in flight while the current stage is multiplied
            load_a(kn);
            compute();
            store_a();
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            buf ^= 1;
        }
        // the item's last stage, with the first one of the next item on its way
        item += G;
        const bool more = item < n_items;
        IgemmItem nx = it;
        if (more) {
            nx = igemm_item<BM, BN>(p, item, G);
            set_rows(nx);
            kc = first_chunk(nx);
            load_b(nx.n0, kc, buf ^ 1);
            load_a(kc);
        }
        compute();
        if (more) {
            store_a();
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // before the results below are stored: those are not waited for
        }
        igemm_join_split<kBK, INAFF>(p, it.m0 + wm * WTM, it.n0 + wn * WTN, next_chunk(it.kc_begin, it.kc_end, ph, pw), it.kc_end,
                                     [&](int k) { return next_chunk(k, it.kc_end, ph, pw); }, [&](int k) { return k * kBK; }, acc, accl);
        igemm_finish<BM, BN, false, STATS>(p, opaque_tid(), wave, acc, it.part, it.m0, it.n0, it.tm, s_stat[0], s_stat[1]);
        if (!more) break;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        it = nx;
        buf ^= 1;
    }
}

// ---- filter gradient -------------------------------------------------------------------------------------------------
// dw[k][j] = sum over pixels of dy[pixel][k] * xcol[pixel][j] with operands split into bf16 terms (see split8): tile BM output channels x
// BN flat filter indices, partial sums over a pixel range, as wgrad_kernel.  Both operands come from memory with the OUTPUT index
// fastest, the matrix instruction wants the reduction index (the pixel) fastest: they are stored to LDS as they come,
// [plane][pixel][index], and read back with the transposing LDS read (lane l of ds_read_b64_tr_b16 receives four pixels of index
// l%16 of a 4 x 16 block).  A pixel's row is padded so that the four rows of 32 indices that half a wavefront reads lie in 64 different banks.
constexpr int wgrad_split_pitch(int b) { return b == 128 ? 160 : 96; }  // 16-bit elements per row: 16 words past a multiple of 64, or 48
typedef short short4v __attribute__((ext_vector_type(4)));
struct Frag8 { short4v lo, hi; };  // eight pixels of one index
__device__ __forceinline__ short4v lds_read_tr(const uint16_t *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(__attribute__((address_space(3))) void *)p);
}

template <int BM, int BN, bool INAFF>
__global__ __launch_bounds__(kConvThreads, wgrad_split_occupancy(BM, BN)) void wgrad_split_kernel(WgradP p)
{
    constexpr int MI = BM / 64, NI = BN / 64;
    constexpr int CA = BM / 4, CB = BN / 4;                                    // 16-byte columns per pixel row
    constexpr int PA = kConvThreads / CA, PB = kConvThreads / CB;              // pixel rows per pass
    constexpr int RA = kBK / PA, RB = kBK / PB;
    constexpr int LA = wgrad_split_pitch(BM), LB = wgrad_split_pitch(BN);
    __shared__ __attribute__((aligned(16))) uint16_t As[3 * kBK * LA];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[3 * kBK * LB];

    const int ntiles = p.tiles_k * p.tiles_j;
    const int item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int split = item / ntiles, tile = item - split * ntiles;
    const int tk = tile / p.tiles_j, tj = tile - tk * p.tiles_j;
    const int k0 = tk * BM, j0 = tj * BN;
    const int pix_begin = split * p.pix_per_split, pix_end = min(p.Mpix, pix_begin + p.pix_per_split);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int ca = tid % CA, pa = tid / CA, cb = tid % CB, pb = tid / CB;

    // filter tap and channel of this thread's four columns (Cin % 4 == 0: they share a tap)
    const int j = j0 + cb * 4;
    const bool jok = j < p.Jdim, kok = k0 + ca * 4 < p.Kout;
    const int r = j / (p.S * p.Cin), rem0 = j - r * (p.S * p.Cin), sx = rem0 / p.Cin, c = rem0 - sx * p.Cin;
    const int th = r - p.pad, tw = sx - p.pad, toff = (th * p.IW + tw) * p.Cin + c;
    float4 in_sc = make_float4(0.f, 0.f, 0.f, 0.f), in_sh = in_sc;
    if (INAFF && jok) {
        in_sc = ldg4(p.in_scale + c);
        in_sh = ldg4(p.in_shift + c);
    }
    // running state of the loads (see wgrad_tile): decoded once, then advanced by kBK pixels per stage
    int apix = pix_begin + pa, bpix = pix_begin + pb, bih[RB], biw[RB];
    unsigned aoff = (unsigned)apix * (unsigned)p.Kout + (unsigned)(k0 + ca * 4), boff[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int pix = bpix + PB * i;
        const int n = (int)fdiv(pix, p.div_ohw), rem = pix - n * (p.OH * p.OW);
        const int oh = (int)fdiv(rem, p.div_ow), ow = rem - oh * p.OW;
        bih[i] = oh * p.stride;
        biw[i] = ow * p.stride;
        boff[i] = ((unsigned)(n * p.IH + bih[i]) * (unsigned)p.IW + (unsigned)biw[i]) * (unsigned)p.Cin;
    }
    float4 ra[RA], rb[RB];
    unsigned in_ok = 0;
    auto load = [&]() {
        const unsigned astep = (unsigned)PA * (unsigned)p.Kout;
#pragma unroll
        for (int i = 0; i < RA; ++i) ra[i] = (kok && apix + PA * i < pix_end) ? ldg4(p.dy + (aoff + astep * i)) : make_float4(0.f, 0.f, 0.f, 0.f);
        in_ok = 0;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int ih = bih[i] + th, iw = biw[i] + tw;
            const bool ok = (bpix + PB * i < pix_end) & jok & ((unsigned)ih < (unsigned)p.IH) & ((unsigned)iw < (unsigned)p.IW);
            rb[i] = ok ? ldg4(p.x + (boff[i] + (unsigned)toff)) : make_float4(0.f, 0.f, 0.f, 0.f);
            if (INAFF && ok) in_ok |= 1u << i;
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
        aoff += p.adv_dy;
    };
    auto put = [&](uint16_t *d, int plane, float4 v, float up) {  // four indices of one pixel; d: the hi plane's place
        v = scaled4(v, up);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const uint32_t w0 = t < 2 ? split_pair(v.x, v.y) : bf16_pack2(v.x, v.y), w1 = t < 2 ? split_pair(v.z, v.w) : bf16_pack2(v.z, v.w);
            *reinterpret_cast<uint2 *>(d + t * plane) = make_uint2(w0, w1);
        }
    };
    auto store = [&]() {
        const float up = split_up();
#pragma unroll
        for (int i = 0; i < RA; ++i) put(&As[(pa + PA * i) * LA + ca * 4], kBK * LA, ra[i], up);
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            if (INAFF && (in_ok & (1u << i))) rb[i] = bn_relu4(rb[i], in_sc, in_sh);  // padding stays zero
            put(&Bs[(pb + PB * i) * LB + cb * 4], kBK * LB, rb[i], up);
        }
    };

    floatx16 acc[MI][NI], accl[MI][NI];
    clear_acc(acc, accl);
    const int frow = 8 * (lane >> 5) + ((lane & 15) >> 2), fcol = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    const uint16_t *fa = &As[frow * LA + wm * (BM / 2) + fcol], *fb = &Bs[frow * LB + wn * (BN / 2) + fcol];
    const int stages = (pix_end - pix_begin + kBK - 1) / kBK;
    load();
    store();
    if (stages > 1) load();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    for (int st = 0; st < stages; ++st) {
        __builtin_amdgcn_s_setprio(1);  // as in wgrad_tile: multiplying goes before address arithmetic, both below the main chain
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            Frag8 af[MI][3], bf[NI][3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const uint16_t *q = fa + (t * kBK + ks * 16) * LA + i * 32;
                    af[i][t] = Frag8{lds_read_tr(q), lds_read_tr(q + 4 * LA)};
                }
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const uint16_t *q = fb + (t * kBK + ks * 16) * LB + i * 32;
                    bf[i][t] = Frag8{lds_read_tr(q), lds_read_tr(q + 4 * LB)};
                }
            }
#pragma unroll
            for (int pr = 0; pr < 6; ++pr) {
                constexpr int ta[6] = {0, 0, 1, 1, 0, 2}, tb[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int n = 0; n < NI; ++n) {
                        floatx16 &d = pr == 0 ? acc[i][n] : accl[i][n];
                        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i][ta[pr]]), __builtin_bit_cast(bf16x8, bf[n][tb[pr]]), d, 0, 0, 0);
                    }
            }
        }
        __builtin_amdgcn_s_setprio(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (st + 1 < stages) {
            store();
            if (st + 2 < stages) load();
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
    }

    const int t2 = opaque_tid(), l2 = t2 & 63;
    float probe = 0.f;  // NaN when a sum is not finite
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int n = 0; n < NI; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc[i][n][e] = (acc[i][n][e] + accl[i][n][e]) * kSplitDown;
                probe = fmaf(acc[i][n][e], 0.f, probe);
            }
    if (__any(probe != probe)) {  // see igemm_join_split
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int n = 0; n < NI; ++n)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][n][e] = 0.f;
        for (int pix = pix_begin + (l2 >> 5); pix < pix_end + (l2 >> 5); pix += 2) {
            const bool in = pix < pix_end;
            const int pq = in ? pix : pix_begin;
            const int n = (int)fdiv(pq, p.div_ohw), rem = pq - n * (p.OH * p.OW);
            const int oh = (int)fdiv(rem, p.div_ow), ow = rem - oh * p.OW;
            float va[MI], vb[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int k = k0 + wm * (BM / 2) + i * 32 + (l2 & 31);
                va[i] = in && k < p.Kout ? p.dy[(size_t)pq * p.Kout + k] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int jj = j0 + wn * (BN / 2) + i * 32 + (l2 & 31);
                const int rr = jj / (p.S * p.Cin), m0 = jj - rr * (p.S * p.Cin), ss = m0 / p.Cin, cc = m0 - ss * p.Cin;
                const int ih = oh * p.stride + rr - p.pad, iw = ow * p.stride + ss - p.pad;
                const bool ok = in && jj < p.Jdim && (unsigned)ih < (unsigned)p.IH && (unsigned)iw < (unsigned)p.IW;
                vb[i] = ok ? p.x[(((size_t)n * p.IH + ih) * p.IW + iw) * p.Cin + cc] : 0.f;
                if (INAFF && ok) vb[i] = fmaxf(fmaf(vb[i], p.in_scale[cc], p.in_shift[cc]), 0.f);
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int nn = 0; nn < NI; ++nn) acc[i][nn] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i], vb[nn], acc[i][nn], 0, 0, 0);
        }
    }
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
