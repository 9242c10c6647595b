// fp32 implicit-GEMM kernels whose filter operand was split into its bf16 terms beforehand (device code; included by
// conv_split.hip).  See split8 in conv_kernels.h for the products and their precision.
//
// What bounds the general kernel (igemm_kernel) once its products run on the bf16 matrix instruction is the vector work of
// splitting: 5.5 instructions per operand element and stage, as many cycles as the matrix work of a 64-wide tile.  The
// filter is the same for every row tile, so here it is split once per call (or once per training step), stored in the
// order and bank swizzle of the LDS image, and copied from memory to LDS without passing through registers.
#pragma once
#include "conv_kernels.h"

namespace rn50 {

constexpr int kPlaneRow = kSplitRow * 4;  // bytes of one filter row's 32 split elements

// w [rows][Kdim] fp32 -> planes [Kdim/32][plane_rows][192 bytes]: stage kc of filter row j as split_chunk lays it out (the
// swizzle depends on j modulo 16 only, so a tile that starts at a multiple of 16 rows is copied to LDS as it is).  Rows from
// `rows` to plane_rows are zeros.  One thread per (stage, row, chunk of eight elements).
struct SplitJob {
    long src_off;   // element offset of the filter from the launch's base
    long dst_off;   // byte offset of its planes
    int rows, plane_rows, kdim, block_begin;
};
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
    const Split8 v = split8(a, b);
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

// The implicit GEMM of igemm_kernel (same work decomposition, MODE 0 and 1, Cin % 32 == 0) with p.planes as filter operand.
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
                if (p.sd == 2) {
                    ok = ok && ((ih | iw) & 1) == 0;
                    ih >>= 1;
                    iw >>= 1;
                } else {
                    ok = ok && (ih % p.sd == 0) && (iw % p.sd == 0);
                    ih /= p.sd;
                    iw /= p.sd;
                }
            }
            ok = ok && ih < p.IH && iw < p.IW;
            const unsigned aoff = (unsigned)(abase[i] + (int)__umul24(__umul24(ih, p.IW) + iw, p.Cin) + c0);
#pragma unroll
            for (int t = 0; t < 2; ++t) ra[i][t] = ok ? ldg4(p.a + (aoff + 16 * t)) : make_float4(0.f, 0.f, 0.f, 0.f);
            if (INAFF && ok) in_ok |= 1u << i;
        }
    };
    auto store_a = [&]() {
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            if (INAFF && (in_ok & (1u << i))) {
                ra[i][0] = bn_relu4(ra[i][0], in_sc[0], in_sh[0]);
                ra[i][1] = bn_relu4(ra[i][1], in_sc[1], in_sh[1]);
            }
            const Split8 v = split8(ra[i][0], ra[i][1]);
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
    int cur_ph = skip_ph, cur_pw = skip_pw;
    load_b(it.n0, kc, 0);
    load_a(kc);
    clear_acc(acc, accl);
    store_a();
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    while (true) {
        int kn = next_chunk(kc + 1, it.kc_end, cur_ph, cur_pw);
        const bool last = kn >= it.kc_end;
        bool more = true;
        IgemmItem nx = it;
        if (last) {
            item += G;
            more = item < n_items;
            if (more) {
                nx = igemm_item<BM, BN>(p, item, G);
                set_rows(nx);
                kn = first_chunk(nx);
            }
        }
        if (more) {  // in flight while the current stage is multiplied
            load_b(nx.n0, kn, buf ^ 1);
            load_a(kn);
        }
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
        if (more) {
            store_a();
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // before the results below are stored: those are not waited for
        }
        if (last) {
            igemm_join_split<kBK, INAFF>(p, it.m0 + wm * WTM, it.n0 + wn * WTN, next_chunk(it.kc_begin, it.kc_end, cur_ph, cur_pw), it.kc_end,
                                         [&](int k) { return next_chunk(k, it.kc_end, cur_ph, cur_pw); }, [&](int k) { return k * kBK; }, acc, accl);
            igemm_finish<BM, BN, false, STATS>(p, acc, it.part, it.m0, it.n0, it.tm, s_stat[0], s_stat[1]);
            if (!more) break;
            clear_acc(acc, accl);
            cur_ph = skip_ph;
            cur_pw = skip_pw;
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        it = nx;
        kc = kn;
        buf ^= 1;
    }
}

// 3x3 convolution of stride 1 and padding 1 (forward, or data gradient with the flipped filter): input and output pixels have
// the same linear index m = (n*H + h)*W + w, and the taps of pixel m are the pixels m + (r-1)*W + (s-1) that lie in the image.
// The general kernel gathers and splits every input element nine times per column tile; here the BM + 2W + 2 pixels under a
// tile's BM pixels go to LDS once per 32 channels, and the nine taps read their fragments from there, a lane whose tap
// falls outside the image from a row of zeros.  Reduction order: stage = (channel block, tap).
// The filter planes come half a stage (16 elements) at a time through a ring of three buffers, two halves ahead of their use.
constexpr int conv3_rows(int bm, int wmax) { return bm + 2 * wmax + 2; }
template <int BM, int BN, int WMAX, bool INAFF, bool STATS>
__global__ __launch_bounds__(kConvThreads, kConv3Occupancy) void conv3x3_kernel(IgemmP p)
{
    constexpr int WTM = BM / 2, WTN = BN / 2, MI = WTM / 32, NI = WTN / 32;
    constexpr int ROWS = conv3_rows(BM, WMAX), SLOTS = (ROWS * 4 + kConvThreads - 1) / kConvThreads;
    constexpr int HB = BN * 6;                  // 16-byte pieces of a filter half stage
    constexpr int NB = HB / kConvThreads;       // ... per thread (BN = 128: 3); BN = 64 takes one piece more for half of the threads
    constexpr int NBX = (HB + kConvThreads - 1) / kConvThreads;
    __shared__ __attribute__((aligned(16))) uint4 Bs[3][HB];
    __shared__ __attribute__((aligned(16))) uint4 As[(ROWS + 1) * 12];  // the last row holds zeros
    __shared__ float s_stat[2][STATS ? BN : 1];
    main_chain_priority();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int W = p.IW, ncb = p.Cin / kBK;
    const int rows = BM + 2 * W + 2;
    const int G = gridDim.x, n_items = p.full_items + p.tail_tiles * p.tail_split;
    int item = blockIdx.x;
    if (item >= n_items) return;
    if (tid < 12) As[ROWS * 12 + tid] = make_uint4(0u, 0u, 0u, 0u);

    // half stage h of a filter stage: of every row the chunks 2h and 2h+1 of each plane.  In memory (and in the LDS image of
    // a whole stage) those sit at chunk positions c ^ (row/4 % 4); the half image is [row][plane][2], chunk 2h + e of a row at
    // e ^ (row/8 % 2) (rows are 24 words long: rows r and r + 8 start in the same bank).
    const unsigned b_lds = lds_offset(&Bs[0][0]) + wave * 1024;
    unsigned b_off[NBX];
#pragma unroll
    for (int u = 0; u < NBX; ++u) {
        const int piece = u * kConvThreads + tid;
        const int row = piece / 6, rem = piece - row * 6;
        const int pos = ((row >> 2) & 2) | ((rem ^ (row >> 3) ^ (row >> 2)) & 1);  // position in its plane for half 0; half 1: pos ^ 2
        b_off[u] = row * kPlaneRow + (rem >> 1) * 64 + pos * 16;
    }
    auto load_b = [&](int n0, int stage, int half, int slot) {
        const int cb = stage / 9, tap = stage - cb * 9;
        const char *src = p.planes + ((size_t)(tap * ncb + cb) * p.plane_rows + n0) * kPlaneRow;
#pragma unroll
        for (int u = 0; u < NBX; ++u)
            if (u < NB || wave < (HB - NB * kConvThreads) / 64) lds_copy16(src, b_off[u] ^ (half * 32), b_lds + slot * (HB * 16) + u * 4096);
    };

    float4 ra[SLOTS][2];
    float4 in_sc[2], in_sh[2];
    unsigned in_ok = 0;
    auto load_a = [&](int m0, int cb) {
        const int c0 = cb * kBK + (tid & 3) * 4;
        if (INAFF) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                in_sc[t] = ldg4(p.in_scale + c0 + 16 * t);
                in_sh[t] = ldg4(p.in_shift + c0 + 16 * t);
            }
            in_ok = 0;
        }
#pragma unroll
        for (int u = 0; u < SLOTS; ++u) {
            const int row = (u * kConvThreads + tid) >> 2;
            const int m = m0 - W - 1 + row;
            const bool ok = row < rows && m >= 0 && m < p.M;
#pragma unroll
            for (int t = 0; t < 2; ++t) ra[u][t] = ok ? ldg4(p.a + ((unsigned)m * (unsigned)p.Cin + c0 + 16 * t)) : make_float4(0.f, 0.f, 0.f, 0.f);
            if (INAFF && ok) in_ok |= 1u << u;
        }
    };
    auto store_a = [&]() {
#pragma unroll
        for (int u = 0; u < SLOTS; ++u) {
            const int row = (u * kConvThreads + tid) >> 2;
            if (row >= rows) continue;
            if (INAFF && (in_ok & (1u << u))) {
                ra[u][0] = bn_relu4(ra[u][0], in_sc[0], in_sh[0]);
                ra[u][1] = bn_relu4(ra[u][1], in_sc[1], in_sh[1]);
            }
            const Split8 v = split8(ra[u][0], ra[u][1]);
            const int at = split_chunk(row, 0, tid & 3);
            As[at] = v.hi;
            As[at + 4] = v.mid;
            As[at + 8] = v.lo;
        }
    };
    // bit 3r+s of taps[i]: tap (r, s) of this lane's pixel of row block i lies in the image
    unsigned taps[MI];
    auto set_taps = [&](const IgemmItem &it) {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int m = it.m0 + wm * WTM + i * 32 + (lane & 31);
            int cls, n, oh, ow;
            decode_row(p, m < p.M ? m : 0, cls, n, oh, ow);
            const unsigned cols = (ow > 0 ? 1u : 0u) | 2u | (ow < W - 1 ? 4u : 0u);
            taps[i] = m < p.M ? (oh > 0 ? cols : 0u) | cols << 3 | (oh < p.IH - 1 ? cols << 6 : 0u) : 0u;
        }
    };

    floatx16 acc[MI][NI], accl[MI][NI];
    IgemmItem it = igemm_item<BM, BN>(p, item, G);
    int st = it.kc_begin, slot = 0;
    load_b(it.n0, st, 0, 0);
    load_b(it.n0, st, 1, 1);
    load_a(it.m0, st / 9);
    set_taps(it);
    clear_acc(acc, accl);
    store_a();
    bool drained = false;
    while (true) {
        // the stage after this one, and whether it needs another input block
        int sn = st + 1;
        const bool last = sn >= it.kc_end;
        bool more = true;
        IgemmItem nx = it;
        if (last) {
            item += G;
            more = item < n_items;
            if (more) {
                nx = igemm_item<BM, BN>(p, item, G);
                sn = nx.kc_begin;
            }
        }
        const bool fresh = more && (last || sn % 9 == 0);
        const int tap = st % 9, tr = tap / 3, ts = tap - 3 * tr;
        // LDS words of this lane's fragments: pixel q's tap is row q + r*W + s of the input block
        int a_row[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int row = wm * WTM + i * 32 + (lane & 31) + tr * W + ts;
            a_row[i] = (taps[i] >> tap) & 1 ? row * 12 + ((lane >> 5) ^ ((row >> 2) & 3)) : ROWS * 12;
        }
        const int b_row = (wn * WTN + (lane & 31)) * 6 + ((lane >> 5) ^ ((lane >> 3) & 1));
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            // this half's filter planes are there when at most the copies of the next half are under way (none are behind the
            // last half; none are left behind a drained wait, whose stores would be waited for here)
            if (!drained) {
                if (half == 1 && !more) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                else if (NB == NBX || wave < (HB - NB * kConvThreads) / 64) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NBX) : "memory");
                else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NB) : "memory");
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            const int ahead = slot >= 1 ? slot - 1 : 2;  // the ring slot two halves on
            if (more) load_b(nx.n0, sn, half, ahead);
            if (half == 0 && fresh) load_a(nx.m0, sn / 9);
            __builtin_amdgcn_s_setprio(3);
            const uint4 *bq = Bs[slot];
            uint4 af[MI][3], bf[NI][3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
#pragma unroll
                for (int i = 0; i < MI; ++i) af[i][t] = As[(a_row[i] ^ (half * 2)) + 4 * t];
#pragma unroll
                for (int j = 0; j < NI; ++j) bf[j][t] = bq[b_row + j * 192 + 2 * t];
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
            __builtin_amdgcn_s_setprio(2);
            slot = slot == 2 ? 0 : slot + 1;
        }
        if (fresh) {
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // every fragment of the input block has been read
            store_a();
        }
        drained = last;
        if (last) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the next stage's planes, before the results below are stored
            igemm_join_split<kBK, INAFF>(p, it.m0 + wm * WTM, it.n0 + wn * WTN, it.kc_begin, it.kc_end, [&](int k) { return k; },
                                         [&](int k) { return ((k % 9) * ncb + k / 9) * kBK; }, acc, accl);
            igemm_finish<BM, BN, false, STATS>(p, acc, it.part, it.m0, it.n0, it.tm, s_stat[0], s_stat[1]);
            if (!more) break;
            clear_acc(acc, accl);
            set_taps(nx);
        }
        it = nx;
        st = sn;
    }
}

}  // namespace rn50
