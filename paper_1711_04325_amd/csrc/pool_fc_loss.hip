// The layers of ResNet-50 (He et al. 2016) around the convolutions: 3x3/2 max pooling, global average
// pooling, the 1000-way fully connected layer and the softmax cross-entropy loss.  NHWC, fp32.
#include "conv_kernels.h"

namespace rn50 {

// one thread per (n, p, q, 4 channels).  INAFF: the pooled tensor is max(0, x*in_scale[c] + in_shift[c]), the BN + ReLU
// in front of the pooling layer applied to every value as it is loaded.
template <class T, bool INAFF>
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(int N, int C4, int H, int W, int P, int Q, const T *__restrict__ x,
                                                          const float *__restrict__ in_scale, const float *__restrict__ in_shift,
                                                          T *__restrict__ y, uint8_t *__restrict__ arg)
{
    // overlapping windows re-read their neighbours' pixels: keep neighbours on one XCD
    const size_t i = (size_t)xcd_contiguous(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (i >= (size_t)N * P * Q * C4) return;
    // 32-bit index arithmetic (the host checks the element count): 64-bit divisions cost more than the nine loads
    const unsigned iu = (unsigned)i;
    const int c = (int)(iu % (unsigned)C4);
    unsigned t = iu / (unsigned)C4;
    const int q = (int)(t % (unsigned)Q);
    t /= (unsigned)Q;
    const int p = (int)(t % (unsigned)P), n = (int)(t / (unsigned)P);
    float best[4] = {0.f, 0.f, 0.f, 0.f};
    int bi[4] = {-1, -1, -1, -1};
    float4 sc = make_float4(0.f, 0.f, 0.f, 0.f), sh = sc;
    if (INAFF) {
        sc = ld4(in_scale, c);
        sh = ld4(in_shift, c);
    }
    // all nine loads first (a tap outside the image loads a clamped pixel and is skipped below), so that they are in
    // flight together
    float4 tap[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const int h = min(max(2 * p + r - 1, 0), H - 1), w = min(max(2 * q + s - 1, 0), W - 1);
            tap[r * 3 + s] = ld4(x, ((size_t)(n * H + h) * W + w) * C4 + c);
        }
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const int h = 2 * p + r - 1, w = 2 * q + s - 1;
            if (h < 0 || h >= H || w < 0 || w >= W) continue;  // padding never wins
            float4 v4 = tap[r * 3 + s];
            if (INAFF)  // the BN + ReLU output as the normalising kernel would have stored it
                v4 = as_stored(y, make_float4(fmaxf(fmaf(v4.x, sc.x, sh.x), 0.f), fmaxf(fmaf(v4.y, sc.y, sh.y), 0.f),
                                              fmaxf(fmaf(v4.z, sc.z, sh.z), 0.f), fmaxf(fmaf(v4.w, sc.w, sh.w), 0.f)));
            const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (bi[e] < 0 || v[e] > best[e]) {  // strict: the first maximal element in window order wins
                    best[e] = v[e];
                    bi[e] = r * 3 + s;
                }
        }
    st4(y, i, make_float4(best[0], best[1], best[2], best[3]));
    reinterpret_cast<uchar4 *>(arg)[i] = make_uchar4((uint8_t)bi[0], (uint8_t)bi[1], (uint8_t)bi[2], (uint8_t)bi[3]);
}

// Gather form: a pixel sums the windows that elected it.  One thread per (n, 2x2 block of pixels, 4 channels): pixel
// (2b + dh, 2a + dw) lies in windows p in {b, b + dh}, q in {a, a + dw}, so the block's four pixels share four windows,
// loaded once (one thread per pixel loads each window up to four times and is bound by the load units, not by memory).
// Each pixel adds its windows in (p, q) order.
template <class T, bool DY2>
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(int N, int C4, int H, int W, int P, int Q, const T *__restrict__ dy,
                                                          const T *__restrict__ dy2, const uint8_t *__restrict__ arg,
                                                          T *__restrict__ dx)
{
    const int HB = (H + 1) / 2, WB = (W + 1) / 2;
    // neighbouring blocks share windows: keep them on one XCD
    const size_t i = (size_t)xcd_contiguous(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (i >= (size_t)N * HB * WB * C4) return;
    const unsigned iu = (unsigned)i;  // 32-bit index arithmetic (the host checks the element count)
    const int c = (int)(iu % (unsigned)C4);
    unsigned t = iu / (unsigned)C4;
    const int wb = (int)(t % (unsigned)WB);
    t /= (unsigned)WB;
    const int hb = (int)(t % (unsigned)HB), n = (int)(t / (unsigned)HB);
    // the four windows (hb + i, wb + j), loaded at clamped positions so that all loads are in flight together
    uchar4 a[4];
    float4 g[4];
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) {
        const int p = min(hb + (t4 >> 1), P - 1), q = min(wb + (t4 & 1), Q - 1);
        const size_t o = ((size_t)(n * P + p) * Q + q) * C4 + c;
        a[t4] = reinterpret_cast<const uchar4 *>(arg)[o];
        g[t4] = ld4(dy, o);
        if (DY2) {
            const float4 g2 = ld4(dy2, o);
            g[t4].x += g2.x; g[t4].y += g2.y; g[t4].z += g2.z; g[t4].w += g2.w;
        }
    }
#pragma unroll
    for (int dh = 0; dh < 2; ++dh)
#pragma unroll
        for (int dw = 0; dw < 2; ++dw) {
            const int h = 2 * hb + dh, w = 2 * wb + dw;
            if (h >= H || w >= W) continue;
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t4 = 0; t4 < 4; ++t4) {
                const int ip = t4 >> 1, iq = t4 & 1;
                if (ip > dh || iq > dw || hb + ip >= P || wb + iq >= Q) continue;  // not a window of this pixel
                const int want = (h - (2 * (hb + ip) - 1)) * 3 + (w - (2 * (wb + iq) - 1));
                if (a[t4].x == want) acc[0] += g[t4].x;
                if (a[t4].y == want) acc[1] += g[t4].y;
                if (a[t4].z == want) acc[2] += g[t4].z;
                if (a[t4].w == want) acc[3] += g[t4].w;
            }
            st4(dx, ((size_t)(n * H + h) * W + w) * C4 + c, make_float4(acc[0], acc[1], acc[2], acc[3]));
        }
}

// Workgroup = 16 float4 columns x 16 slices of the H*W positions; the slice sums are added in pairs, pairs of pairs, ... (error of
// 49 positive values against 64 bits 5.2e-8, in slice order 6.9e-8).  A thread has up to four positions in flight: with 4 slices of 13 positions one after
// the other the 32 x 7 x 7 x 2048 tensor took 6.6 us, with this cut 4.4 - 5.0.
constexpr int kAvgCols = 16, kAvgSlices = 16;
template <class T>
__global__ __launch_bounds__(kAvgCols * kAvgSlices) void avgpool_fwd_kernel(int N, int C4, int HW, const T *__restrict__ x, float *__restrict__ y)
{
    __shared__ float4 red[kAvgSlices][kAvgCols];
    const int cl = threadIdx.x % kAvgCols, slice = threadIdx.x / kAvgCols;
    const int c = blockIdx.x * kAvgCols + cl, n = blockIdx.y;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < C4)
        for (int j0 = slice; j0 < HW; j0 += 4 * kAvgSlices) {
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = ld4(x, ((size_t)n * HW + min(j0 + u * kAvgSlices, HW - 1)) * C4 + c);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (j0 + u * kAvgSlices < HW) {
                    s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w;
                }
        }
    red[slice][cl] = s;
    __syncthreads();
    if (slice == 0 && c < C4) {
        float4 v[kAvgSlices];
#pragma unroll
        for (int t = 0; t < kAvgSlices; ++t) v[t] = red[t][cl];
#pragma unroll
        for (int half = kAvgSlices / 2; half; half /= 2)
#pragma unroll
            for (int t = 0; t < half; ++t) v[t] = make_float4(v[t].x + v[t + half].x, v[t].y + v[t + half].y, v[t].z + v[t + half].z, v[t].w + v[t + half].w);
        s = v[0];
        const float inv = 1.0f / (float)HW;
        reinterpret_cast<float4 *>(y)[(size_t)n * C4 + c] = make_float4(s.x * inv, s.y * inv, s.z * inv, s.w * inv);
    }
}

template <class T>
__global__ __launch_bounds__(256) void avgpool_bwd_kernel(int N, int C4, int HW, const float *__restrict__ dy, T *__restrict__ dx)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)N * HW * C4) return;
    const unsigned iu = (unsigned)i;  // 32-bit index arithmetic (the host checks the element count)
    const int c = (int)(iu % (unsigned)C4);
    const int n = (int)(iu / ((unsigned)HW * (unsigned)C4));
    const float4 g = ld4(dy, (size_t)n * C4 + c);
    const float inv = 1.0f / (float)HW;
    st4(dx, i, make_float4(g.x * inv, g.y * inv, g.z * inv, g.w * inv));
}

// ---- fully connected layer -----------------------------------------------------------------------------------------------
// Forward and data gradient: 16 x 16 outputs per workgroup of 16 wavefronts, on the matrix cores with split operands (see split8 in
// conv_kernels.h), operands straight from memory in fragment order.  A wavefront takes every 16th step of 32 reduction elements; the 16
// partial tiles meet in LDS and are added in pairs, pairs of pairs, ... (2048 features of one sign, relative error against 64 bits 3.5e-8, one
// after the other 6.2e-8).  Such small calls are bound by the latency of their loads: with tiles of
// 32 x 32 the 1000 classes of 32 samples fill 32 of the 256 CUs and take 19.7 us, with these 10.9 (the vector kernel, which read all features
// once per class, 28.7); the data gradient 18.4 and 10.7 (16.2).
constexpr int kFcWaves = 16, kFcTile = 16, kFcStep = 32;
typedef float floatx4 __attribute__((ext_vector_type(4)));
struct FcFrag { float4 lo, hi; };  // eight reduction elements of one row: lane l has row l % 16, elements 8 * (l / 16) of the step

// Adds the wavefronts' tiles; thread t of the first 256 returns the sum of output (t / 16, t % 16).
__device__ inline float fc_join(const floatx4 &acc, const floatx4 &accl, float (*red)[kFcTile * kFcTile])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][(4 * (lane >> 4) + e) * kFcTile + (lane & 15)] = (acc[e] + accl[e]) * kSplitDown;
    __syncthreads();
    float s = 0.f;
    if (threadIdx.x < kFcTile * kFcTile) {
        float v[kFcWaves];
#pragma unroll
        for (int w = 0; w < kFcWaves; ++w) v[w] = red[w][threadIdx.x];
#pragma unroll
        for (int half = kFcWaves / 2; half; half /= 2)
#pragma unroll
            for (int w = 0; w < half; ++w) v[w] += v[w + half];
        s = v[0];
    }
    return s;
}
// U: steps whose loads are in flight together
template <int U, class LoadA, class LoadB>
__device__ __forceinline__ void fc_products(int steps, LoadA load_a, LoadB load_b, floatx4 &acc, floatx4 &accl)
{
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = accl[e] = 0.f;
    for (int s0 = wave; s0 < steps; s0 += kFcWaves * U) {
        FcFrag a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {  // steps past the end load zeros
            a[u] = load_a(s0 + u * kFcWaves);
            b[u] = load_b(s0 + u * kFcWaves);
        }
        const float up = split_up();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const Split8 sa = split8(a[u].lo, a[u].hi, up), sb = split8(b[u].lo, b[u].hi, up);
            const uint4 ta[3] = {sa.hi, sa.mid, sa.lo}, tb[3] = {sb.hi, sb.mid, sb.lo};
            constexpr int ia[6] = {0, 0, 1, 1, 0, 2}, ib[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
            for (int pr = 0; pr < 6; ++pr) {
                floatx4 &d = pr == 0 ? acc : accl;
                d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ta[ia[pr]]), __builtin_bit_cast(bf16x8, tb[ib[pr]]), d, 0, 0, 0);
            }
        }
    }
}

// y[n,k] = <f[n,:], w[k,:]> + b[k].  J % 4 == 0.
__global__ __launch_bounds__(64 * kFcWaves) void fc_fwd_kernel(int N, int J, int K, const float *__restrict__ f, const float *__restrict__ w,
                                                              const float *__restrict__ b, float *__restrict__ y)
{
    __shared__ float red[kFcWaves][kFcTile * kFcTile];
    const int lane = threadIdx.x & 63;
    const int k0 = blockIdx.x * kFcTile, n0 = blockIdx.y * kFcTile;
    // rows past the end repeat the last one and are never stored
    const float *fr = f + (size_t)min(n0 + (lane & 15), N - 1) * J, *wr = w + (size_t)min(k0 + (lane & 15), K - 1) * J;
    auto row = [&](const float *p, int step) {
        const int j = step * kFcStep + (lane >> 4) * 8;
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        return FcFrag{j < J ? ldg4(p + j) : z, j + 4 < J ? ldg4(p + j + 4) : z};
    };
    floatx4 acc, accl;
    fc_products<4>((J + kFcStep - 1) / kFcStep, [&](int st) { return row(fr, st); }, [&](int st) { return row(wr, st); }, acc, accl);
    float s = fc_join(acc, accl, red);
    const int n = n0 + threadIdx.x / kFcTile, k = k0 + threadIdx.x % kFcTile;
    if (threadIdx.x >= kFcTile * kFcTile || n >= N || k >= K) return;
    if (!isfinite(s)) {  // an infinite operand has no finite split: this output in plain fp32
        s = 0.f;
        for (int j = 0; j < J; ++j) s = fmaf(f[(size_t)n * J + j], w[(size_t)k * J + j], s);
    }
    y[(size_t)n * K + k] = s + b[k];
}

// df[n,j] = sum_k dy[n,k] w[k,j]
__global__ __launch_bounds__(64 * kFcWaves) void fc_bwd_data_kernel(int N, int J, int K, const float *__restrict__ w, const float *__restrict__ dy,
                                                                   float *__restrict__ df)
{
    __shared__ float red[kFcWaves][kFcTile * kFcTile];
    const int lane = threadIdx.x & 63;
    const int j0 = blockIdx.x * kFcTile, n0 = blockIdx.y * kFcTile;
    const float *gr = dy + (size_t)min(n0 + (lane & 15), N - 1) * K, *wc = w + min(j0 + (lane & 15), J - 1);
    auto column = [&](const float *p, long stride, int step) {
        const int k = step * kFcStep + (lane >> 4) * 8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = k + e < K ? p[(k + e) * stride] : 0.f;
        return FcFrag{make_float4(v[0], v[1], v[2], v[3]), make_float4(v[4], v[5], v[6], v[7])};
    };
    floatx4 acc, accl;
    fc_products<2>((K + kFcStep - 1) / kFcStep, [&](int st) { return column(gr, 1, st); }, [&](int st) { return column(wc, J, st); }, acc, accl);
    float s = fc_join(acc, accl, red);
    const int n = n0 + threadIdx.x / kFcTile, j = j0 + threadIdx.x % kFcTile;
    if (threadIdx.x >= kFcTile * kFcTile || n >= N || j >= J) return;
    if (!isfinite(s)) {
        s = 0.f;
        for (int k = 0; k < K; ++k) s = fmaf(dy[(size_t)n * K + k], w[(size_t)k * J + j], s);
    }
    df[(size_t)n * J + j] = s;
}

// dw[k,j] = sum_n dy[n,k] f[n,j]; db[k] = sum_n dy[n,k], samples in order.  A thread takes four columns of four classes, a workgroup
// 64 column groups x 16 classes; bound by the latency of its loads, so those of 32 samples are in flight together and dy comes
// through LDS: 32 x 2048 x 1000 in 8.8 us (one class per thread, eight samples in flight: 14.0).
constexpr int kFcClasses = 4, kFcSamples = 32;
__global__ __launch_bounds__(256) void fc_bwd_weight_kernel(int N, int J4, int K, const float *__restrict__ f, const float *__restrict__ dy,
                                                            float *__restrict__ dw, float *__restrict__ db)
{
    __shared__ float g[kFcSamples][4 * kFcClasses];
    const int j = blockIdx.x * 64 + (threadIdx.x & 63), wave = threadIdx.x >> 6;
    const int kb = blockIdx.y * 4 * kFcClasses, k0 = kb + wave * kFcClasses;
    const int jl = min(j, J4 - 1);
    float4 acc[kFcClasses];
    float sb[kFcClasses];
#pragma unroll
    for (int c = 0; c < kFcClasses; ++c) {
        acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        sb[c] = 0.f;
    }
    for (int nb = 0; nb < N; nb += kFcSamples) {
        float4 fv[kFcSamples];
#pragma unroll
        for (int u = 0; u < kFcSamples; ++u) fv[u] = ld4(f, (size_t)min(nb + u, N - 1) * J4 + jl);
        __syncthreads();  // the chunk before has been read
#pragma unroll
        for (int t = 0; t < kFcSamples * 4 * kFcClasses / 256; ++t) {
            const int i = threadIdx.x + 256 * t, n = i / (4 * kFcClasses), k = i % (4 * kFcClasses);
            g[n][k] = nb + n < N && kb + k < K ? dy[(size_t)(nb + n) * K + kb + k] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kFcSamples; ++u)
            if (nb + u < N) {
#pragma unroll
                for (int c = 0; c < kFcClasses; ++c) {
                    const float gv = g[u][wave * kFcClasses + c];
                    acc[c].x = fmaf(gv, fv[u].x, acc[c].x); acc[c].y = fmaf(gv, fv[u].y, acc[c].y);
                    acc[c].z = fmaf(gv, fv[u].z, acc[c].z); acc[c].w = fmaf(gv, fv[u].w, acc[c].w);
                    sb[c] += gv;
                }
            }
    }
    if (j >= J4) return;
#pragma unroll
    for (int c = 0; c < kFcClasses; ++c)
        if (k0 + c < K) {
            reinterpret_cast<float4 *>(dw)[(size_t)(k0 + c) * J4 + j] = acc[c];
            if (j == 0) db[k0 + c] = sb[c];
        }
}

// Single workgroup of 16 wavefronts; each wavefront takes rows wave, wave+16, ...  Row losses are summed in row order.  Bound by the
// exponentials of one CU: one per element, the probabilities are those divided by their sum (32 x 1000: 11.4 -> 10.2 us).
constexpr int kSoftmaxRegs = 16;  // rows of up to 1024 classes are held in registers
__global__ __launch_bounds__(1024) void softmax_ce_kernel(int N, int K, const float *__restrict__ logits, const int32_t *__restrict__ labels,
                                                          float *__restrict__ loss, float *__restrict__ dlogits)
{
    __shared__ float row_loss[1024];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float invN = 1.0f / (float)N;
    for (int n = wave; n < N; n += 16) {
        const float *z = logits + (size_t)n * K;
        const int lab = labels[n];
        // a label outside [0, K) makes the loss NaN (and puts no one-hot term into the gradient); z[lab] is never read for it
        const bool lab_ok = (unsigned)lab < (unsigned)K;
        const float zl = lab_ok ? z[lab] : 0.f;  // on its way with the row
        if (K <= 64 * kSoftmaxRegs) {
            // the row fits in registers: one round of loads in flight instead of three dependent passes over memory
            float v[kSoftmaxRegs];
#pragma unroll
            for (int i = 0; i < kSoftmaxRegs; ++i) v[i] = lane + 64 * i < K ? z[lane + 64 * i] : -INFINITY;
            float mx = v[0];
#pragma unroll
            for (int i = 1; i < kSoftmaxRegs; ++i) mx = fmaxf(mx, v[i]);
            mx = wave_max(mx);
            float se = 0.f;
#pragma unroll
            for (int i = 0; i < kSoftmaxRegs; ++i) {
                v[i] = lane + 64 * i < K ? expf(v[i] - mx) : 0.f;
                se += v[i];
            }
            se = wave_sum(se);
            const float lse = mx + logf(se), inv = 1.0f / se;
#pragma unroll
            for (int i = 0; i < kSoftmaxRegs; ++i) {
                const int k = lane + 64 * i;
                if (k < K) dlogits[(size_t)n * K + k] = (v[i] * inv - (k == lab ? 1.f : 0.f)) * invN;
            }
            if (lane == 0) row_loss[n] = lab_ok ? lse - zl : __builtin_nanf("");
            continue;
        }
        float mx = -INFINITY;
        for (int k = lane; k < K; k += 64) mx = fmaxf(mx, z[k]);
        mx = wave_max(mx);
        float se = 0.f;
        for (int k = lane; k < K; k += 64) se += expf(z[k] - mx);
        se = wave_sum(se);
        const float lse = mx + logf(se);
        for (int k = lane; k < K; k += 64) dlogits[(size_t)n * K + k] = (expf(z[k] - lse) - (k == lab ? 1.f : 0.f)) * invN;
        if (lane == 0) row_loss[n] = lab_ok ? lse - zl : __builtin_nanf("");
    }
    __syncthreads();
    if (wave == 0) {
        float s = 0.f;
        for (int nb = 0; nb < N; nb += 64) {  // from registers: one LDS read for 64 rows instead of one behind the other
            const float v = nb + lane < N ? row_loss[nb + lane] : 0.f;
            const int cnt = min(64, N - nb);
            for (int t = 0; t < cnt; ++t) s += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), t));
        }
        if (lane == 0) loss[0] = s * invN;
    }
}

static int dims_check(const char *who, int n, int c, int h, int w)
{
    RN50_REQUIRE(n > 0 && c > 0 && h > 0 && w > 0, RN50_EINVAL, "%s: non-positive dimension", who);
    RN50_REQUIRE(c % 4 == 0, RN50_EUNSUPPORTED, "%s: channel count must be a multiple of 4", who);
    RN50_REQUIRE((long)n * h * w * c < (1L << 31), RN50_EUNSUPPORTED, "%s: tensor too large", who);
    return RN50_OK;
}

}  // namespace rn50

using namespace rn50;

template <class T>
static int maxpool_fwd_impl(const char *who, int n, int c, int h, int w, const T *x, const float *in_scale, const float *in_shift,
                            T *y, uint8_t *argidx, void *stream)
{
    if (int rc = dims_check(who, n, c, h, w)) return rc;
    RN50_REQUIRE(x && y && argidx, RN50_EINVAL, "%s: null pointer", who);
    RN50_REQUIRE(aligned16(x) && aligned16(y) && aligned16(argidx) && aligned16(in_scale) && aligned16(in_shift), RN50_EINVAL,
                 "%s: pointers must be 16-byte aligned", who);
    RN50_REQUIRE((in_scale != nullptr) == (in_shift != nullptr), RN50_EINVAL, "%s: scale and shift go together", who);
    const int P = (h - 1) / 2 + 1, Q = (w - 1) / 2 + 1;
    const size_t total = (size_t)n * P * Q * (c / 4);
    RN50_REQUIRE((size_t)n * h * w * (c / 4) < (1ull << 31), RN50_EUNSUPPORTED, "%s: more than 2^31 groups of four channels", who);
    if (in_scale)
        hipLaunchKernelGGL((maxpool_fwd_kernel<T, true>), dim3(ceil_div(total, 256)), dim3(256), 0, (hipStream_t)stream, n, c / 4, h, w, P, Q, x,
                           in_scale, in_shift, y, argidx);
    else
        hipLaunchKernelGGL((maxpool_fwd_kernel<T, false>), dim3(ceil_div(total, 256)), dim3(256), 0, (hipStream_t)stream, n, c / 4, h, w, P, Q, x,
                           in_scale, in_shift, y, argidx);
    return launch_status(who);
}

extern "C" int maxpool3x3s2_fwd(int n, int c, int h, int w, const float *x, float *y, uint8_t *argidx, void *stream)
{
    return maxpool_fwd_impl<float>("maxpool3x3s2_fwd", n, c, h, w, x, nullptr, nullptr, y, argidx, stream);
}

extern "C" int maxpool3x3s2_fwd_bnrelu_input(int n, int c, int h, int w, const float *x, const float *in_scale, const float *in_shift,
                                             float *y, uint8_t *argidx, void *stream)
{
    RN50_REQUIRE(in_scale && in_shift, RN50_EINVAL, "maxpool3x3s2_fwd_bnrelu_input: null scale or shift");
    return maxpool_fwd_impl<float>("maxpool3x3s2_fwd_bnrelu_input", n, c, h, w, x, in_scale, in_shift, y, argidx, stream);
}

extern "C" int maxpool3x3s2_fwd_bf16(int n, int c, int h, int w, const uint16_t *x, const float *in_scale_or_null,
                                     const float *in_shift_or_null, uint16_t *y, uint8_t *argidx, void *stream)
{
    return maxpool_fwd_impl<bf16_t>("maxpool3x3s2_fwd_bf16", n, c, h, w, x, in_scale_or_null, in_shift_or_null, y, argidx, stream);
}

template <class T>
static int maxpool_bwd_impl(const char *who, int n, int c, int h, int w, const T *dy, const T *dy2_or_null, const uint8_t *argidx, T *dx,
                            void *stream)
{
    if (int rc = dims_check(who, n, c, h, w)) return rc;
    RN50_REQUIRE(dy && dx && argidx, RN50_EINVAL, "%s: null pointer", who);
    RN50_REQUIRE(aligned16(dy) && aligned16(dy2_or_null) && aligned16(dx) && aligned16(argidx), RN50_EINVAL,
                 "%s: pointers must be 16-byte aligned", who);
    const int P = (h - 1) / 2 + 1, Q = (w - 1) / 2 + 1;
    RN50_REQUIRE((size_t)n * h * w * (c / 4) < (1ull << 31), RN50_EUNSUPPORTED, "%s: more than 2^31 groups of four channels", who);
    const size_t total = (size_t)n * ((h + 1) / 2) * ((w + 1) / 2) * (c / 4);  // one thread per 2x2 block of pixels
    if (dy2_or_null)
        hipLaunchKernelGGL((maxpool_bwd_kernel<T, true>), dim3(ceil_div(total, 256)), dim3(256), 0, (hipStream_t)stream, n, c / 4, h, w, P, Q, dy,
                           dy2_or_null, argidx, dx);
    else
        hipLaunchKernelGGL((maxpool_bwd_kernel<T, false>), dim3(ceil_div(total, 256)), dim3(256), 0, (hipStream_t)stream, n, c / 4, h, w, P, Q, dy,
                           dy2_or_null, argidx, dx);
    return launch_status(who);
}

extern "C" int maxpool3x3s2_bwd(int n, int c, int h, int w, const float *dy, const float *dy2_or_null, const uint8_t *argidx,
                                float *dx, void *stream)
{
    return maxpool_bwd_impl<float>("maxpool3x3s2_bwd", n, c, h, w, dy, dy2_or_null, argidx, dx, stream);
}

extern "C" int maxpool3x3s2_bwd_bf16(int n, int c, int h, int w, const uint16_t *dy, const uint16_t *dy2_or_null, const uint8_t *argidx,
                                     uint16_t *dx, void *stream)
{
    return maxpool_bwd_impl<bf16_t>("maxpool3x3s2_bwd_bf16", n, c, h, w, dy, dy2_or_null, argidx, dx, stream);
}

template <class T>
static int avgpool_fwd_impl(const char *who, int n, int c, int h, int w, const T *x, float *y, void *stream)
{
    if (int rc = dims_check(who, n, c, h, w)) return rc;
    RN50_REQUIRE(x && y && aligned16(x) && aligned16(y), RN50_EINVAL, "%s: null or misaligned pointer", who);
    hipLaunchKernelGGL((avgpool_fwd_kernel<T>), dim3(ceil_div(c / 4, kAvgCols), n), dim3(kAvgCols * kAvgSlices), 0, (hipStream_t)stream, n,
                       c / 4, h * w, x, y);
    return launch_status(who);
}

template <class T>
static int avgpool_bwd_impl(const char *who, int n, int c, int h, int w, const float *dy, T *dx, void *stream)
{
    if (int rc = dims_check(who, n, c, h, w)) return rc;
    RN50_REQUIRE(dy && dx && aligned16(dy) && aligned16(dx), RN50_EINVAL, "%s: null or misaligned pointer", who);
    RN50_REQUIRE((size_t)n * h * w * (c / 4) < (1ull << 31), RN50_EUNSUPPORTED, "%s: more than 2^31 groups of four channels", who);
    hipLaunchKernelGGL((avgpool_bwd_kernel<T>), dim3(ceil_div((long)n * h * w * c / 4, 256)), dim3(256), 0, (hipStream_t)stream, n, c / 4, h * w, dy, dx);
    return launch_status(who);
}

extern "C" int avgpool_fwd(int n, int c, int h, int w, const float *x, float *y, void *stream)
{
    return avgpool_fwd_impl<float>("avgpool_fwd", n, c, h, w, x, y, stream);
}
extern "C" int avgpool_bwd(int n, int c, int h, int w, const float *dy, float *dx, void *stream)
{
    return avgpool_bwd_impl<float>("avgpool_bwd", n, c, h, w, dy, dx, stream);
}
extern "C" int avgpool_fwd_bf16(int n, int c, int h, int w, const uint16_t *x, float *y, void *stream)
{
    return avgpool_fwd_impl<bf16_t>("avgpool_fwd_bf16", n, c, h, w, x, y, stream);
}
extern "C" int avgpool_bwd_bf16(int n, int c, int h, int w, const float *dy, uint16_t *dx, void *stream)
{
    return avgpool_bwd_impl<bf16_t>("avgpool_bwd_bf16", n, c, h, w, dy, dx, stream);
}

extern "C" int fc_fwd(int n, int j, int k, const float *f, const float *w, const float *b, float *y, void *stream)
{
    RN50_REQUIRE(n > 0 && j > 0 && k > 0, RN50_EINVAL, "fc_fwd: non-positive dimension");
    RN50_REQUIRE(j % 4 == 0, RN50_EUNSUPPORTED, "fc_fwd: input width must be a multiple of 4");
    RN50_REQUIRE(f && w && b && y && aligned16(f) && aligned16(w) && aligned16(b) && aligned16(y), RN50_EINVAL,
                 "fc_fwd: null or misaligned pointer");
    hipLaunchKernelGGL(fc_fwd_kernel, dim3(ceil_div(k, kFcTile), ceil_div(n, kFcTile)), dim3(64 * kFcWaves), 0, (hipStream_t)stream, n, j, k, f, w, b, y);
    return launch_status("fc_fwd");
}

extern "C" int fc_bwd(int n, int j, int k, const float *f, const float *w, const float *dy, float *df, float *dw, float *db,
                      void *stream)
{
    RN50_REQUIRE(n > 0 && j > 0 && k > 0, RN50_EINVAL, "fc_bwd: non-positive dimension");
    RN50_REQUIRE(j % 4 == 0, RN50_EUNSUPPORTED, "fc_bwd: input width must be a multiple of 4");
    RN50_REQUIRE(f && w && dy && df && dw && db, RN50_EINVAL, "fc_bwd: null pointer");
    RN50_REQUIRE(aligned16(f) && aligned16(w) && aligned16(dy) && aligned16(df) && aligned16(dw) && aligned16(db), RN50_EINVAL,
                 "fc_bwd: pointers must be 16-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(fc_bwd_weight_kernel, dim3(ceil_div(j / 4, 64), ceil_div(k, 4 * kFcClasses)), dim3(256), 0, st, n, j / 4, k, f, dy, dw, db);
    hipLaunchKernelGGL(fc_bwd_data_kernel, dim3(ceil_div(j, kFcTile), ceil_div(n, kFcTile)), dim3(64 * kFcWaves), 0, st, n, j, k, w, dy, df);
    return launch_status("fc_bwd");
}

extern "C" int softmax_ce(int n, int k, const float *logits, const int32_t *labels, float *loss, float *dlogits, void *stream)
{
    RN50_REQUIRE(n > 0 && k > 0, RN50_EINVAL, "softmax_ce: non-positive dimension");
    RN50_REQUIRE(n <= 1024, RN50_EUNSUPPORTED, "softmax_ce: at most 1024 rows");
    RN50_REQUIRE(logits && labels && loss && dlogits, RN50_EINVAL, "softmax_ce: null pointer");
    hipLaunchKernelGGL(softmax_ce_kernel, dim3(1), dim3(1024), 0, (hipStream_t)stream, n, k, logits, labels, loss, dlogits);
    return launch_status("softmax_ce");
}
