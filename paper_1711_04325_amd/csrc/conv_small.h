// Implicit GEMM for calls that do not fill the chip (device code; included by conv_small.hip): fp32 operands on the fp32 matrix instruction.
//
// What bounded the general kernel there is a chain: tiles of 64 x 64 leave most CUs idle unless the reduction is cut over workgroups, whose partial tiles
// a second launch then adds (2.4 us at the least), and a piece's stages pass one after the other through registers, LDS and two barriers.  Here the
// reduction is cut over the wavefronts of one workgroup: each loads its fragments straight from memory (the operands are in the caches), all of several
// stages in flight at once, and the partial tiles meet in LDS, where the sum's statistics are gathered as well.
#pragma once
#include "conv_kernels.h"

namespace rn50 {

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ const float4 g_zero4 = {0.f, 0.f, 0.f, 0.f};  // what lanes outside the image load

constexpr int kSmallWaves = 4;  // 8 and 16 were as fast where one workgroup runs on a CU, and slower (up to twice) where more do

// A workgroup: TM x TN blocks of 16 rows x 16 columns; wavefront w takes the stages of 32 reduction elements w, w + 4, ..., each in four sums (a single block
// in eight): the matrix instruction's results follow each other at their full rate, and a sum has a 16th or 32nd of the reduction: errors against 64
// bits are 0.4 - 1 times those of the pieces and their ordered sum before.
// Cin % 32 == 0 (a stage stays inside one filter tap), Nout % 4 == 0, R*S <= 32, no dilation.  FLIP: the filter of a data gradient as it is, [k][tap][row].
// INAFF: see IgemmP.  STATS: the output's statistics per TM * 16 rows as well.
template <int TM, int TN, bool FLIP, bool INAFF, bool STATS>
__global__ __launch_bounds__(64 * kSmallWaves) void igemm_small_kernel(IgemmWideP p)
{
    constexpr int W = kSmallWaves, U = TM + TN == 2 ? 4 : TM + TN == 3 ? 3 : 2;  // stages in flight
    __shared__ floatx4 red[W][TM * TN * 64];
    main_chain_priority();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), pl = lane & 15, g = lane >> 4;
    const int tile = xcd_contiguous(blockIdx.x, gridDim.x);
    // each XCD takes a range of rows or of columns, whichever leaves its L2 less to fetch
    const bool by_row = (long)p.M * p.Cin >= (long)p.Nout * p.Kdim;
    const int tq = tile / (by_row ? p.tiles_n : p.tiles_m), tr = tile - tq * (by_row ? p.tiles_n : p.tiles_m);
    const int tm = by_row ? tq : tr, m0 = tm * (TM * 16), n0 = (by_row ? tr : tq) * (TN * 16);

    // rows of the gathered tensor under this lane's pixels, and which filter taps lie inside the image
    int base[TM];
    unsigned mask[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + i * 16 + pl;
        base[i] = 0;
        mask[i] = 0;
        if (m < p.M) {
            int cls, n, oh, ow;
            decode_row(p, m, cls, n, oh, ow);
            const int ih = oh * p.so + p.off, iw = ow * p.so + p.off;
            unsigned bit = 1;
            for (int r = 0; r < p.R; ++r)
                for (int s = 0; s < p.S; ++s, bit <<= 1)
                    if ((unsigned)(ih + r) < (unsigned)p.IH && (unsigned)(iw + s) < (unsigned)p.IW) mask[i] |= bit;
            base[i] = ((n * p.IH + ih) * p.IW + iw) * p.Cin + 4 * g;  // below 2^31 where a tap is inside
        }
    }
    bool col_in[TN];
    const float *wrow[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = n0 + j * 16 + pl;
        col_in[j] = col < p.Nout;
        wrow[j] = p.b + (FLIP ? (long)(col_in[j] ? col : 0) + (long)(4 * g) * p.flip_taps * p.Nout : (long)(col_in[j] ? col : 0) * p.Kdim + 4 * g);
    }
    constexpr int SUMS = TM * TN == 1 ? 8 : 4;
    floatx4 acc[SUMS][TM][TN];
#pragma unroll
    for (int e = 0; e < SUMS; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[e][i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int stages = p.Kdim / kBK;
    for (int st0 = wave; st0 < stages; st0 += W * U) {
        float4 a[U][TM][2], b[U][TN][2];
        float4 sc[INAFF ? U : 1][2], sh[INAFF ? U : 1][2];
        unsigned in[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int st = st0 + u * W, k0 = min(st, stages - 1) * kBK;
            const bool live = st < stages;  // past the end: zeros on both sides
            const int tap = (int)fdiv(k0, p.div_cin), c0 = k0 - tap * p.Cin;
            const int r = (int)fdiv(tap, p.div_s), s = tap - r * p.S;
            const int off = (r * p.IW + s) * p.Cin + c0;
            in[u] = 0;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const bool ok = live && (mask[i] >> tap & 1);
                in[u] |= (unsigned)ok << i;
                const float *q = p.a + (unsigned)(base[i] + off);
#pragma unroll
                for (int h = 0; h < 2; ++h) a[u][i][h] = *reinterpret_cast<const float4 *>(ok ? q + 16 * h : reinterpret_cast<const float *>(&g_zero4));
            }
            if (INAFF) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    sc[u][h] = ldg4(p.in_scale + c0 + 4 * g + 16 * h);
                    sh[u][h] = ldg4(p.in_shift + c0 + 4 * g + 16 * h);
                }
            }
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (FLIP) {
                        const long step = (long)p.flip_taps * p.Nout;
                        const float *q = wrow[j] + (long)(c0 + 16 * h) * step + (long)(p.flip_taps - 1 - tap) * p.Nout;
                        b[u][j][h] = make_float4(q[0], q[step], q[2 * step], q[3 * step]);
                    } else {
                        b[u][j][h] = ldg4(wrow[j] + k0 + 16 * h);
                    }
                    if (!live) b[u][j][h] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
        }
        __builtin_amdgcn_sched_barrier(0);  // every load on its way before the first product
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (INAFF) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        if (in[u] >> i & 1) a[u][i][h] = bn_relu4(a[u][i][h], sc[u][h], sh[u][h]);  // padding stays zero
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            acc[(e + 4 * h) % SUMS][i][j] =
                                __builtin_amdgcn_mfma_f32_16x16x4f32((&b[u][j][h].x)[e], (&a[u][i][h].x)[e], acc[(e + 4 * h) % SUMS][i][j], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int e = 4; e < SUMS; ++e) acc[e - 4][i][j] += acc[e][i][j];
            red[wave][(i * TN + j) * 64 + lane] = (acc[0][i][j] + acc[1][i][j]) + (acc[2][i][j] + acc[3][i][j]);
        }
    __syncthreads();
    if (wave >= TN) return;  // wavefront j: the blocks of column block j
    const int j = wave, col = n0 + j * 16 + 4 * g;
    floatx4 v[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const floatx4 *r = &red[0][(i * TN + j) * 64 + lane];
        v[i] = (r[0] + r[TM * TN * 64]) + (r[2 * TM * TN * 64] + r[3 * TM * TN * 64]);
    }
    if (STATS) {
        const int valid = min(TM * 16, p.M - m0);
        float4 mean, m2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float sum = 0.f, dev = 0.f;
#pragma unroll
            for (int i = 0; i < TM; ++i) sum += i * 16 + pl < valid ? v[i][e] : 0.f;
            const float mu = row16_sum(sum) / (float)valid;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const float d = v[i][e] - mu;
                dev = i * 16 + pl < valid ? fmaf(d, d, dev) : dev;
            }
            (&mean.x)[e] = mu;
            (&m2.x)[e] = row16_sum(dev);
        }
        if (pl == 0 && col < p.Nout) {
            *reinterpret_cast<float4 *>(&p.stat_mean[(long)tm * p.Nout + col]) = mean;
            *reinterpret_cast<float4 *>(&p.stat_m2[(long)tm * p.Nout + col]) = m2;
        }
    }
    if (col >= p.Nout) return;  // Nout % 4 == 0: the four columns are inside together
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + i * 16 + pl;
        if (m >= p.M) continue;
        const long row = out_row_index(p, m), at = row * p.Nout + col;
        *reinterpret_cast<floatx4 *>(&p.out[at]) = v[i];
        if (p.scatter2 == 1) {
            const floatx4 z = {0.f, 0.f, 0.f, 0.f};
            *reinterpret_cast<floatx4 *>(&p.out[at + p.Nout]) = z;
            *reinterpret_cast<floatx4 *>(&p.out[at + 2l * p.OW * p.Nout]) = z;
            *reinterpret_cast<floatx4 *>(&p.out[at + (2l * p.OW + 1) * p.Nout]) = z;
        }
    }
}

}  // namespace rn50
