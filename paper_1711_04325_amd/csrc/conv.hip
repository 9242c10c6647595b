// Host side of the convolution entry points: validation, tile/split selection, workspace layout, launches.
#include <algorithm>

#include "conv_kernels.h"

namespace rn50 {

int conv_check(const char *who, const rn50_conv_desc *d)
{
    RN50_REQUIRE(d, RN50_EINVAL, "%s: null descriptor", who);
    RN50_REQUIRE(d->n > 0 && d->c > 0 && d->h > 0 && d->w > 0 && d->k > 0 && d->r > 0 && d->s > 0 && d->stride > 0 && d->pad >= 0,
                 RN50_EINVAL, "%s: non-positive dimension", who);
    RN50_REQUIRE(d->layout == RN50_LAYOUT_NHWC, RN50_EUNSUPPORTED, "%s: only the NHWC/KRSC layout has kernels", who);
    RN50_REQUIRE(d->in_dtype == RN50_DTYPE_F32 || d->in_dtype == RN50_DTYPE_BF16 || d->in_dtype == RN50_DTYPE_BF16_ACT ||
                     d->in_dtype == RN50_DTYPE_BF16_ACT_F32IN,
                 RN50_EUNSUPPORTED, "%s: unknown operand dtype", who);
    RN50_REQUIRE(d->h + 2 * d->pad >= d->r && d->w + 2 * d->pad >= d->s, RN50_EINVAL, "%s: filter larger than the padded input", who);
    RN50_REQUIRE(d->pad < d->r && d->pad < d->s, RN50_EUNSUPPORTED, "%s: padding must be smaller than the filter", who);
    RN50_REQUIRE((long)d->h * d->w < (1L << 24) && d->c < (1 << 24) && d->k < (1 << 24), RN50_EUNSUPPORTED,
                 "%s: H*W, C and K must be below 2^24 (24-bit multiplies in the gather)", who);
    const long P = (d->h + 2 * d->pad - d->r) / d->stride + 1, Q = (d->w + 2 * d->pad - d->s) / d->stride + 1;
    RN50_REQUIRE((long)d->n * d->h * d->w * d->c < (1L << 31) && (long)d->n * P * Q * d->k < (1L << 31) &&
                     (long)d->n * d->h * d->w < (1L << 27) && (long)d->k * d->r * d->s * d->c < (1L << 31),
                 RN50_EUNSUPPORTED, "%s: tensor too large for 32-bit indexing", who);
    return RN50_OK;
}

// Storage of the activation tensors a call reads and writes: 0 fp32, 1 bfloat16 bits, 2 bfloat16 bits except the layer
// input x, which is fp32 (the network's first layer).  Both bf16 forms multiply on the bf16 MFMA.
static int act_of(const rn50_conv_desc *d)
{
    return d->in_dtype == RN50_DTYPE_BF16_ACT ? 1 : d->in_dtype == RN50_DTYPE_BF16_ACT_F32IN ? 2 : 0;
}
static bool bf16_of(const rn50_conv_desc *d) { return d->in_dtype != RN50_DTYPE_F32; }
// Reduction elements per LDS stage of the implicit GEMM: 64 for bf16 operands through the vector gather when a stage of 64 stays
// inside one filter tap (cin = channels of the gathered tensor), else 32.
static int igemm_bk(bool bf16, int act, int cin) { return bf16 && act != 2 && cin % (2 * kBK) == 0 ? 2 * kBK : kBK; }

struct Geom { int P, Q; long Mout, Min; int Kdim; };
static Geom geom(const rn50_conv_desc *d)
{
    Geom g;
    g.P = (d->h + 2 * d->pad - d->r) / d->stride + 1;
    g.Q = (d->w + 2 * d->pad - d->s) / d->stride + 1;
    g.Mout = (long)d->n * g.P * g.Q;
    g.Min = (long)d->n * d->h * d->w;
    g.Kdim = d->r * d->s * d->c;
    return g;
}

// ---- tile and split selection ------------------------------------------------------------------------
constexpr double kCUs = 256.0;
constexpr double kBytesPerClk = 8e12 / 2.4e9;  // HBM bytes per core clock, whole chip
constexpr double kLaunchClks = 6000.0;         // one extra kernel launch, in core clocks

struct GemmPlan { int bm, bn, split, chunks_per_split; bool products = false, terms = false; };  // products: of split operands (wgrad_split_kernel)

// Kernel of a forward or data-gradient call: the general implicit GEMM, or one that takes the filter prepared beforehand: split into bf16
// terms (igemm_pre_kernel, fp32 operands) or rounded to bf16 (igemm_act_kernel, bf16 activations).
enum IgemmKind { kGeneral = 0, kPre = 1, kAct = 2, kHalf = 3, kSmall = 4 };
static int igemm_kind_occupancy(int kind, int bm, int bn)
{
    return kind == kHalf ? half_occupancy(bm, bn) : kind == kPre ? igemm_pre_occupancy(bm, bn) : kind == kAct ? igemm_act_occupancy(bm, bn) : igemm_occupancy(bm, bn);
}

// Plans measured on the MI355X for the ResNet-50 layer shapes: {op, n, c, h, k, r, stride, pad, bm, bn, split}.
// Other shapes use the cost model below.
static const PlanRow kTuned[] = {
#include "conv_plans.inc"
    {-1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}};
// The same for bf16 activations in memory, where most layers are bound by memory traffic and other tiles win; consulted first
// for that storage (shapes it does not list fall through to the table above).
static const PlanRow kTunedAct[] = {
#include "conv_plans_bf16act.inc"
    {-1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}};

static bool plan_matches(const PlanRow &t, const rn50_conv_desc *d, int op)
{
    return t.op == op && t.n == d->n && t.c == d->c && t.h == d->h && d->w == d->h && t.k == d->k && t.r == d->r && d->s == d->r &&
           t.stride == d->stride && t.pad == d->pad;
}

// Rows set with rn50_set_option("plan_overrides") go before the table (a tuning aid: plans tried inside a whole step).
static bool override_plan(const Config &cfg, const rn50_conv_desc *d, int op, GemmPlan *pl)
{
    for (const PlanRow &t : cfg.overrides)
        if (plan_matches(t, d, op)) {
            pl->bm = t.bm; pl->bn = t.bn; pl->split = t.split;
            return true;
        }
    return false;
}
static bool tuned_plan(const Config &cfg, const rn50_conv_desc *d, int op, GemmPlan *pl)
{
    if (override_plan(cfg, d, op, pl)) return true;
    if (cfg.no_tuned) return false;
    if (act_of(d))
        for (const PlanRow &t : kTunedAct)
            if (plan_matches(t, d, op)) {
                pl->bm = t.bm; pl->bn = t.bn; pl->split = t.split;
                return true;
            }
    for (const PlanRow &t : kTuned)
        if (plan_matches(t, d, op)) {
            pl->bm = t.bm; pl->bn = t.bn; pl->split = t.split;
            return true;
        }
    return false;
}

static bool forced_plan(bool has, const int v[3], GemmPlan *pl)
{
    if (!has) return false;
    pl->bm = v[0]; pl->bn = v[1]; pl->split = v[2];
    return true;
}

static double tile_eff(int bm, int bn) { return bm == 128 && bn == 128 ? 1.0 : (bm == 64 && bn == 64 ? 0.72 : 0.86); }

// Persistent implicit-GEMM launch: G workgroups; the first full_items tiles whole, the last tail_tiles tiles cut
// into tail_split pieces of tail_chunks reduction chunks each.
struct IgemmPlan { int kind, bm, bn, grid, full_items, tail_tiles, tail_split, tail_chunks; size_t ws_floats; bool products = false; size_t prep_bytes = 0; double cost = 0; };  // products: of split operands (kGeneral); prep_bytes: workspace of the operands prepared by the call; cost: model_plan's


static IgemmPlan make_igemm_plan(int kind, int bm, int bn, long M, int Nout, int kchunks, int want_split, bool allow_split)
{
    IgemmPlan pl;
    pl.kind = kind; pl.bm = bm; pl.bn = bn;
    const int tiles = ceil_div(M, bm) * ceil_div(Nout, bn);
    const int Gmax = (int)kCUs * igemm_kind_occupancy(kind, bm, bn);
    pl.full_items = tiles / Gmax * Gmax;
    pl.tail_tiles = tiles - pl.full_items;
    int sp = allow_split ? want_split : 1;
    if (sp > kchunks) sp = kchunks;
    if (sp < 1) sp = 1;
    pl.tail_chunks = ceil_div(kchunks, sp);
    pl.tail_split = pl.tail_tiles ? ceil_div(kchunks, pl.tail_chunks) : 1;
    const int items = pl.full_items + pl.tail_tiles * pl.tail_split;
    pl.grid = pl.full_items ? Gmax : std::min(Gmax, (items + 7) / 8 * 8);
    pl.ws_floats = pl.tail_split > 1 ? (size_t)pl.tail_tiles * pl.tail_split * bm * bn : 0;
    return pl;
}

// modelled time in core clocks (of the fp32 instruction; the general split kernel is planned with it as well, for want of a model of its own: 5 % off
// the best plan on average)
static double igemm_cost(const IgemmPlan &pl, int kchunks, double chunk_clks)
{
    const int occ = igemm_kind_occupancy(pl.kind, pl.bm, pl.bn);
    const double full_rounds = pl.full_items / (kCUs * occ);
    double t = full_rounds * occ * (kchunks + 2.0) * chunk_clks;
    if (pl.tail_tiles) {
        const double pieces = (double)pl.tail_tiles * pl.tail_split;
        const double per_cu = ceil(pieces / kCUs);
        t += per_cu * (pl.tail_chunks + 3.0) * chunk_clks / (per_cu >= 2.0 ? 1.0 : 0.65);
        if (pl.tail_split > 1) t += kLaunchClks + (pl.tail_split + 1.0) * pl.tail_tiles * pl.bm * pl.bn * 4.0 / kBytesPerClk;
    }
    return t;
}
// The same for igemm_pre_kernel, in microseconds: per tile shape the time of a 32-element stage while a CU is full, the time
// of an item beyond its stages, and the time of a stage of a workgroup that has a CU to itself.  Fitted to 5,000 measured launches (226
// calls of 140 shapes, each with every tile and several splits): the plan it picks takes 4.6 % longer than the best one measured on
// average, 13 % at the 90th percentile.
static double igemm_pre_cost(const IgemmPlan &pl, int kchunks)
{
    static const double c128x128[3] = {1.212, 2.258, 1.714}, c128x64[3] = {0.755, 1.278, 1.090}, c64x128[3] = {0.705, 2.072, 1.058},
                        c64x64[3] = {0.400, 0.733, 0.872};
    const double *c = pl.bm == 128 ? (pl.bn == 128 ? c128x128 : c128x64) : (pl.bn == 128 ? c64x128 : c64x64);
    const int occ = igemm_pre_occupancy(pl.bm, pl.bn);
    double t = pl.full_items / (kCUs * occ) * occ * (kchunks * c[0] + c[1]);
    if (pl.tail_tiles) {
        const double per_cu = ceil((double)pl.tail_tiles * pl.tail_split / kCUs);
        t += std::max(per_cu * (pl.tail_chunks * c[0] + c[1]), pl.tail_chunks * c[2] + 4.35);
        if (pl.tail_split > 1) t += 3.1 + (pl.tail_split + 1.0) * pl.tail_tiles * pl.bm * pl.bn * 4.0 / 5.8e6;
    }
    return t;
}

// The same for igemm_half_kernel, without its preparation.  Fitted to 1,554 measured launches (86 calls, every tile, seven splits): the plan it picks
// takes 1.5 % longer than the best one measured on average, 5 % at the 90th percentile.
static double igemm_half_cost(const IgemmPlan &pl, int kchunks)
{
    static const double c128x64[3] = {0.364, 1.301, 0.642}, c64x128[3] = {0.331, 0.771, 0.566}, c64x64[3] = {0.195, 0.464, 0.473};
    const double *c = pl.bm == 128 ? c128x64 : pl.bn == 128 ? c64x128 : c64x64;
    const int occ = half_occupancy(pl.bm, pl.bn);
    double t = pl.full_items / (kCUs * occ) * occ * (kchunks * c[0] + c[1]);
    if (pl.tail_tiles) {
        const double per_cu = ceil((double)pl.tail_tiles * pl.tail_split / kCUs);
        t += std::max(per_cu * (pl.tail_chunks * c[0] + c[1]), pl.tail_chunks * c[2]);
        if (pl.tail_split > 1) t += 3.1 + (pl.tail_split + 1.0) * pl.tail_tiles * pl.bm * pl.bn * 4.0 / 5.8e6;
    }
    return t;
}

// The same for igemm_act_kernel (kchunks: stages of 64); a forward pass with its statistics and their merge, which reads a row of partials per row tile.
// Fitted to 5,100 measured launches (166 calls of 130 shapes, every tile, up to seven splits): the plan it picks takes 1.0 % longer than the best one
// measured in forward passes, 2.3 % in data gradients, on average.  The rows of the measured table, which igemm_act_kernel took before, are those of the
// general kernel: 7.7 % longer (64 -> 256 channels at 56x56, N = 256, forward 215 us in tiles of 64 x 128, 180 in 128 x 128; 1024 -> 512 at 14x14, N = 32: 42, 25).
// A row stays all the same where the model gains less than this many microseconds: the launches it was fitted to repeat a call on operands that are in the
// caches, and few large tiles wait longest for those that are not.  3x3 256 -> 256 at 14x14, N = 32, forward: 28.3 us in 200 workgroups of 64 x 128, 30.1 in
// 496 pieces of 128 x 128; in a step 4 us the other way round.  Step with bf16 activations, rows alone / model alone / margin of 1.5, 2.5, 3.5, 4.5, 6, 8:
// N = 32 4.62, 4.73 / 4.71, 4.67, 4.64, 4.62, 4.62, 4.63 ms; v1.5 4.90, 4.89 / 4.88, 4.85, 4.82, 4.81, 4.83, 4.84; N = 256 21.71, 21.24 / 21.22, 21.23, 21.17,
// 21.23, 21.34, 21.43.
constexpr double kActRowMargin = 4.0;
static double igemm_act_cost(const IgemmPlan &pl, bool fwd, long M, int Nout, int kchunks)
{
    static const double f128x128[3] = {0.519, 0.965, 0.625}, f128x64[3] = {0.336, 0.585, 0.393}, f64x128[3] = {0.307, 0.0, 0.347}, f64x64[3] = {0.198, 0.051, 0.230};
    static const double b128x128[3] = {0.516, 1.405, 0.633}, b128x64[3] = {0.319, 0.800, 0.399}, b64x128[3] = {0.288, 0.788, 0.483}, b64x64[3] = {0.192, 0.401, 0.402};
    const double *c = pl.bm == 128 ? (pl.bn == 128 ? (fwd ? f128x128 : b128x128) : (fwd ? f128x64 : b128x64))
                                   : (pl.bn == 128 ? (fwd ? f64x128 : b64x128) : (fwd ? f64x64 : b64x64));
    const int occ = igemm_act_occupancy(pl.bm, pl.bn);
    double t = pl.full_items / (kCUs * occ) * occ * (kchunks * c[0] + c[1]);
    if (pl.tail_tiles) {
        const double per_cu = ceil((double)pl.tail_tiles * pl.tail_split / kCUs);
        t += std::max(per_cu * (pl.tail_chunks * c[0] + c[1]), pl.tail_chunks * c[2] + (fwd ? 1.7 : 4.9));
        if (pl.tail_split > 1) t += (pl.tail_split + 1.0) * pl.tail_tiles * pl.bm * pl.bn * 4.0 / 5.0e6;
    }
    const double bands = ceil_div(M, pl.bm);
    return fwd ? t + 0.0042 * bands + 3.4e-5 * bands * Nout : t;
}

static IgemmPlan model_plan(int kind, long M, int Nout, int kchunks, int bk, bool allow_split, int max_bm = 128, bool fwd = true)
{
    IgemmPlan best{};
    double best_cost = 1e300;  // left in best.cost
    static const int splits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
    for (int bm = max_bm; bm >= 64; bm -= 64)
        for (int bn = 128; bn >= 64; bn -= 64) {
            if (bn == 128 && Nout <= 64) continue;
            if (bm == 128 && M <= 64) continue;
            if (kind == kHalf && bm == 128 && bn == 128) continue;  // no registers for its three sets of sums
            for (int sp : splits) {
                if (sp > 1 && (!allow_split || kchunks / sp < 2)) break;
                const IgemmPlan pl = make_igemm_plan(kind, bm, bn, M, Nout, kchunks, sp, allow_split);
                const double cost = kind == kHalf ? igemm_half_cost(pl, kchunks) : kind == kPre ? igemm_pre_cost(pl, kchunks)
                                                 : kind == kAct ? igemm_act_cost(pl, fwd, M, Nout, kchunks)
                                                 : igemm_cost(pl, kchunks, 4096.0 * (bk / (double)kBK) * (bm * bn / 16384.0) / tile_eff(bm, bn));
                if (cost < best_cost) { best_cost = cost; best = pl; }
            }
        }
    best.cost = best_cost;
    return best;
}

// data gradient of a 1x1 stride-2 convolution on an even-sized input: a GEMM whose rows are scattered
static bool is_scatter2(const rn50_conv_desc *d)
{
    return d->r == 1 && d->s == 1 && d->stride == 2 && d->pad == 0 && d->h % 2 == 0 && d->w % 2 == 0;
}

constexpr int kActStage = 64;          // channels of igemm_act_kernel's stage
// Preparing a filter for one call costs a launch (3 us and more with a large filter), which the faster kernel earns back on calls long
// enough: measured prepared / general over 40 shapes, fp32 0.72-0.99 of the speed below 5 GFLOP, at 5-10 0.98-1.14 with reductions of
// 1024 and more and 0.95-1.05 with shorter ones, 1.01-1.05 above; bf16 activations 0.77-0.99 below 4, 0.95-1.16 at 4-9, 1.00-1.15 above.  Where many filters are prepared in one launch only the
// smallest calls (fewer rows than eight tiles) keep the general kernel.
constexpr long kPlanesMinRows = 1024;
constexpr double kPlanesMinFlops = 5e9, kPlanesMinFlopsF32 = 1e10;  // the latter for fp32 reductions shorter than 1024

// The network's first layer (fp32, or an fp32 image in front of bf16 activations), which has kernels of its own (tiles of 8 x 16 pixels)
static bool stem_layer(const rn50_conv_desc *d)
{
    return d->c == 3 && d->r == 7 && d->s == 7 && d->stride == 2 && d->pad == 3 && d->k == 64 &&
           (d->in_dtype == RN50_DTYPE_F32 || d->in_dtype == RN50_DTYPE_BF16_ACT_F32IN) && (long)d->n * d->h * d->w * 3 < (1l << 31) &&
           !config()->no_stem_kernel;
}

// What a call with less workspace than its query names runs: without the halves; below that without any preparation.
static Fp32Math less_room(Fp32Math math) { return math == kFp32Split ? kNoHalf : kNoPlanes; }
// Operands as fp16 halves (conv_half.h) where that is as precise as the call's other plan, whose sums of `piece` elements are the longest.
// Relative error against 64 bits, halves / bf16 terms (90 calls): forward behind a ReLU 1.07 - 1.26e-7 whatever the length, with terms 0.9 - 1.2e-7 in
// pieces of 300 - 650 elements, 1.24e-7 in 768, 1.43e-7 in 1024, 1.5e-7 in 1152; data gradients 1.11 - 1.31e-7, with terms 1.47e-7 in 512,
// 1.55e-7 in 576, 2.1e-7 in 1152 (1.2 - 1.5e-7 in 384).  What the halves drop stays where most of an operand is zeros, the roundings of a long sum do not:
// with 80, 90, 97 % zeros in either operand 1.04 - 1.18e-7, 0.97 - 1.12e-7, 0.88 - 1.04e-7, with terms 0.87 - 1.06e-7, 0.69 - 0.82e-7, 0.45 - 0.6e-7 (14 calls);
// in data gradients in pieces of 512 with 50 % already (1.14e-7, 0.98e-7).  The option half_products is for such operands.  A line at 700 for data
// gradients as well: the step at N = 32 9.42 -> 9.63 ms.
static bool half_as_precise(bool fwd, double piece) { return piece >= (fwd ? 700 : 480); }
// Preparing both operands (two launches and one more gap than the other plan has; the gathered tensor is read twice and written once), in microseconds;
// what the other plan takes beyond igemm_pre_cost: the filter's preparation, in a data gradient its flip.
static double half_prep_cost(double elems) { return 14.75 + 2.28e-6 * elems; }
static double pre_extra_cost(bool fwd, bool given) { return given ? 3.0 : fwd ? 6.0 : 10.0; }
constexpr double kHalfMinFlops = 1e9;
// Workspace of their preparation: [exponents][shares of the largest magnitude][marks][filter][gathered tensor]
constexpr int kHalfShares = 512;
struct HalfRoom { size_t part, marks, planes, halves, total; int nmarks; };
static HalfRoom half_room(long pixels, int cin, int rows, int kdim)
{
    HalfRoom r;
    size_t cur = 256;
    auto take = [&](size_t b) { const size_t o = cur; cur += (b + 255) / 256 * 256; return o; };
    r.part = take(2 * kHalfShares * 4);
    r.nmarks = 1 + (int)((pixels >> kHalfMarkShift) + 1) + rows;
    r.marks = take((size_t)r.nmarks * 4);
    r.planes = take((size_t)(kdim / kBK) * plane_rows_of(rows) * 128);
    r.halves = take((size_t)pixels * cin * 4 + 256);  // zeros ahead of it
    r.total = cur;
    return r;
}

// out[M][Nout] with reduction length Kdim (in elements)
// cin: channels of the gathered tensor (the forward pass gathers x, the data gradient dy)
// given: the call comes with its filter prepared
static IgemmPlan plan_igemm_kind(const rn50_conv_desc *d, int op, long M, int Nout, int Kdim, bool allow_split, int cin, Fp32Math math, bool given)
{
    const int bk = igemm_bk(bf16_of(d), act_of(d), cin);
    const int kchunks = ceil_div(Kdim, bk);
    GemmPlan pl;
    const std::shared_ptr<const Config> cfg = config();
    const bool split = (math == kFp32Split || math == kNoHalf) && !bf16_of(d) && !(op == RN50_OP_FWD && stem_layer(d));  // (the first layer: what its query names)
    auto as_split = [&](IgemmPlan g) {
        g.products = split;
        return g;
    };
    if (forced_plan(cfg->has_igemm_plan, cfg->igemm_plan, &pl) || override_plan(*cfg, d, op, &pl))
        return as_split(make_igemm_plan(kGeneral, pl.bm, pl.bn, M, Nout, kchunks, pl.split, allow_split));
    // the dilated gather of a strided data gradient needs registers that a 128-row tile does not leave (igemm_pre_kernel spills)
    const bool dilated = op == RN50_OP_BWD_DATA && d->stride == 2 && !is_scatter2(d);
    const double flops = 2.0 * M * Nout * Kdim;
    const bool geometry = M >= kPlanesMinRows && (op == RN50_OP_FWD || d->stride <= 2) && math != kNoPlanes &&
                          (given || flops >= (split && Kdim < 1024 ? kPlanesMinFlopsF32 : kPlanesMinFlops));
    const bool fwd = op == RN50_OP_FWD;
    const long gathered = fwd ? (long)d->n * d->h * d->w : geom(d).Mout;
    if (split && math != kNoHalf && !dilated && cin % kBK == 0 && Nout % 4 == 0 && (fwd || d->stride <= 2) && d->r * d->s <= 32 && gathered * cin < (1l << 30) - 64) {
        IgemmPlan half{};
        for (const PlanRow &t : cfg->operand_plans)
            if (plan_matches(t, d, op) && (t.bm == 64 || t.bn == 64)) half = make_igemm_plan(kHalf, t.bm, t.bn, M, Nout, kchunks, t.split, allow_split);
        bool pre_row = false;  // a row for igemm_pre_kernel goes before the choice below
        for (const PlanRow &t : cfg->pre_plans) pre_row |= geometry && plan_matches(t, d, op);
        if (!half.grid && !pre_row && (cfg->half_products & (fwd ? 1 : 2)) && M >= kPlanesMinRows && flops >= kHalfMinFlops) {
            const IgemmPlan other = plan_igemm_kind(d, op, M, Nout, Kdim, allow_split, cin, kNoHalf, given);
            if (!half_as_precise(fwd, other.full_items || other.tail_split < 2 ? Kdim : (double)Kdim / other.tail_split)) return other;
            half = model_plan(kHalf, M, Nout, kchunks, bk, allow_split);
            // right in 79 of 83 calls measured both ways, the others within 9 %
            if (half.cost + half_prep_cost((double)gathered * cin) >= 0.95 * (model_plan(kPre, M, Nout, kchunks, bk, allow_split).cost + pre_extra_cost(fwd, given)))
                return other;
        }
        if (half.grid) {
            half.prep_bytes = half_room(gathered, cin, Nout, Kdim).total;
            return half;
        }
    }
    if (split && geometry && cin % kBK == 0) {
        for (const PlanRow &t : cfg->pre_plans)
            if (plan_matches(t, d, op) && (!dilated || t.bm == 64))
                return make_igemm_plan(kPre, t.bm, t.bn, M, Nout, kchunks, t.split, allow_split);
        return model_plan(kPre, M, Nout, kchunks, bk, allow_split, dilated ? 64 : 128);
    }
    if (act_of(d) == 1 && geometry && cin % kActStage == 0) {
        for (const PlanRow &t : cfg->pre_plans)
            if (plan_matches(t, d, op)) return make_igemm_plan(kAct, t.bm, t.bn, M, Nout, kchunks, t.split, allow_split);
        const IgemmPlan own = model_plan(kAct, M, Nout, kchunks, bk, allow_split, 128, fwd);
        if (!tuned_plan(*cfg, d, op, &pl)) return own;
        const IgemmPlan row = make_igemm_plan(kAct, pl.bm, pl.bn, M, Nout, kchunks, pl.split, allow_split);
        return igemm_act_cost(row, fwd, M, Nout, kchunks) <= own.cost + kActRowMargin ? row : own;
    }
    const IgemmPlan general = tuned_plan(*cfg, d, op, &pl) ? make_igemm_plan(kGeneral, pl.bm, pl.bn, M, Nout, kchunks, pl.split, allow_split)
                                                            : model_plan(kGeneral, M, Nout, kchunks, bk, allow_split);
    // fp32 operands split as they are loaded pay where the matrix unit has work: with more than one workgroup on a CU (time on the fp32
    // instruction / split, 110 shapes of 0.001 - 11 GFLOP: 0.94-0.98 with fewer, 1.02-1.6 with more), and where channels are gathered one by
    // one, with 128-row tiles (1.00-1.12, with 64-row tiles 0.87-1.01).  Below that the shorter kernel wins.
    if (split && general.grid > (int)kCUs && (cin % kBK == 0 || general.bm == 128)) return as_split(model_plan(kGeneral, M, Nout, kchunks, bk, allow_split));
    return general;
}

static IgemmPlan plan_igemm(const rn50_conv_desc *d, int op, long M, int Nout, int Kdim, bool allow_split, int cin, Fp32Math math, bool given)
{
    IgemmPlan pl = plan_igemm_kind(d, op, M, Nout, Kdim, allow_split, cin, math, given);
    if (pl.kind == kPre || pl.kind == kAct) pl.prep_bytes = given ? 0 : filter_planes_bytes(Nout, Kdim, pl.kind == kAct);
    return pl;
}

// igemm_small_kernel for a call of fp32 operands whose plan is `other` (grid 0: it stays with that).  It needs no workspace; a call needs what its query
// names all the same.  beside: microseconds that the other way takes beyond its launches (the filter's flip).
// Modelled times of both, in microseconds, from 220 calls of 0.006 - 3 GFLOP, forward and data gradients.
// Calls with split operands stay (0.2 GFLOP and more; half the error).
// stat_room: bytes for the statistics of its row tiles (0: the call takes none); a tile whose statistics need more is not taken, so that the workspace
// that a call asks for, and refuses to go without, is that of its other plan.
constexpr double kFlipLaunch = 3.5;
static IgemmPlan plan_small(const rn50_conv_desc *d, int op, long M, int Nout, int Kdim, int cin, const IgemmPlan &other, double beside, size_t stat_room = 0)
{
    auto fits = [&](int bm) { return !stat_room || (size_t)2 * ceil_div(M, bm) * Nout * sizeof(float) <= stat_room; };
    IgemmPlan s{};
    const std::shared_ptr<const Config> cfg = config();
    const double gflop = 2e-9 * M * Nout * Kdim;
    if (bf16_of(d) || cin % kBK || Nout % 4 || d->r * d->s > 32 || other.kind != kGeneral || cfg->has_igemm_plan ||
        (op == RN50_OP_BWD_DATA && d->stride > 1 && !is_scatter2(d)))
        return s;
    s.kind = kSmall;
    s.tail_split = 1;
    auto set = [&](int bm, int bn) {
        s.bm = bm; s.bn = bn;
        s.full_items = s.grid = ceil_div(M, bm) * ceil_div(Nout, bn);
    };
    for (const PlanRow &t : cfg->small_plans)
        if (plan_matches(t, d, op)) {  // whatever it needs: plan_fwd_stats makes room
            set(t.bm, t.bn);
            return s;
        }
    if (gflop > 1.0 || other.products || !cfg->overrides.empty()) return s;
    // the other way: with an ordered sum, or one launch (its reduction is short then)
    double best = 0.9 * (beside + (other.tail_split > 1 ? 7.2 + 0.0018 * Kdim + 12.0 * std::max(0.0, gflop - 0.1) : 5.6 + 0.012 * std::min(Kdim, 256) + 8.0 * gflop));
    for (int bm = 16; bm <= 32; bm += 16)
        for (int bn = 16; fits(bm) && bn <= 32; bn += 16) {
            const int blocks = bm * bn / 256, per_cu = ceil_div((long)ceil_div(M, bm) * ceil_div(Nout, bn), (int)kCUs);
            const double t = blocks == 1 ? 2.1 + per_cu * (0.8 + 0.0037 * Kdim) : blocks == 2 ? 2.3 + per_cu * (0.9 + 0.0055 * Kdim) : 2.6 + per_cu * (1.4 + 0.0085 * Kdim);
            if (t * (d->r > 1 ? 1.15 : 1.0) < best) {
                best = t * (d->r > 1 ? 1.15 : 1.0);
                set(bm, bn);
            }
        }
    return s;
}

// The filter-gradient kernels take two stages per trip of their loop: a range of an odd number of stages ends with a stage of
// zeros, so ranges are cut at even counts where there is more than one range.
static int even_stages(int cps, int pchunks) { return cps < pchunks ? cps + (cps & 1) : cps; }

// dw[Kout][Jdim] with the reduction over Mpix pixels, split into `split` ranges of chunks_per_split stages
static GemmPlan plan_wgrad_any_tile(const rn50_conv_desc *d, int Kout, int Jdim, long Mpix, Fp32Math math);

// Whether a filter gradient over `pixels` is as precise with split operands in `ranges` ranges as on the fp32 instruction in `unit` ranges.
// The fp32 instruction rounds the sum of a range every two pixels, the bf16 instruction every 16, but that one drops low bits of products
// that are small beside others of the 16, towards zero.  Behind a BN's backward pass and a ReLU half of the products are small and of
// one sign, and what is dropped of them does not fall with the length of a range.  Relative error E against 64 bits for such operands,
// measured for 26 shapes of 6,272 to 65,536 pixels: E^2 / pixels is 2.1 - 3.0e-16 / unit on the fp32 instruction and 4.5e-17 / ranges +
// 2.6e-18 + 3.2e-23 pixels with split operands.  (Over 401,408 pixels, 3x3 64 x 64: 6.6e-7 in 224 ranges, split 1.6e-6 however cut.)
// Where all products have one sign both fall with 1 / ranges, and the split's is that of 2.3 times as many.
// The sides of the line: 128 -> 512, 50,176 pixels 4.9e-7 in 61 ranges, split in 61 5.0e-7 (not split); 3x3 128 x 128, 50,176 pixels 4.5e-7 in
// 56, split in 112 4.1e-7 (split); 3x3 256 x 256, 25,088 pixels 4.3e-7 in 28, split in 7 4.7e-7 and in 16 3.5e-7 (split in 13 or more).
// Speed alone would split them all (3x3 64 x 64, 100,352 pixels: 1.3 times).
static bool wgrad_split_as_precise(long pixels, int unit, int ranges)
{
    return 4.5e-17 / ranges + 2.6e-18 + 3.2e-23 * pixels <= 2.6e-16 / unit && ranges * 2.3 >= unit;
}

static GemmPlan plan_wgrad(const rn50_conv_desc *d, int Kout, int Jdim, long Mpix, Fp32Math math)
{
    GemmPlan pl = plan_wgrad_any_tile(d, Kout, Jdim, Mpix, math);
    if (act_of(d) && (pl.bm != 64 || pl.bn != 64)) {
        // the bf16-activation kernel has 64x64 tiles only: as many workgroups as the chosen plan by a matching split
        const int pchunks = ceil_div(Mpix, kBK);
        const long wgs = (long)ceil_div(Kout, pl.bm) * ceil_div(Jdim, pl.bn) * pl.split;
        int split = std::max(1, (int)(wgs / ((long)ceil_div(Kout, 64) * ceil_div(Jdim, 64))));
        if (split > pchunks) split = pchunks;
        pl.bm = pl.bn = 64;
        pl.chunks_per_split = even_stages(ceil_div(pchunks, split), pchunks);
        pl.split = ceil_div(pchunks, pl.chunks_per_split);
    }
    return pl;
}

// Modelled time of wgrad_split_kernel and its ordered sum in microseconds: per tile shape the time of a 32-pixel stage while a CU is full, the
// time of a work item beyond its stages, and the time of a stage of workgroups that do not fill a CU.  Fitted to 124 calls with every
// tile and up to seven splits; the plan it picks takes 1.2 % longer than the best one measured on average, 4 % at the 90th percentile.
static double wgrad_split_cost(int bm, int bn, int Kout, int Jdim, int split, int cps)
{
    static const double c128x128[3] = {1.383, 2.172, 1.929}, c128x64[3] = {0.793, 0.692, 1.123}, c64x128[3] = {0.822, 0.797, 1.279},
                        c64x64[3] = {0.470, 0.147, 0.729};
    const double *c = bm == 128 ? (bn == 128 ? c128x128 : c128x64) : (bn == 128 ? c64x128 : c64x64);
    const int per_cu = ceil_div((long)ceil_div(Kout, bm) * ceil_div(Jdim, bn) * split, (int)kCUs);
    return std::max(per_cu * (cps * c[0] + c[1]), ceil_div(per_cu, wgrad_split_occupancy(bm, bn)) * (cps * c[2] + 0.71)) +
           (split + 1.0) * Kout * Jdim * 4.0 / 7.94e6;
}

// The same for wgrad_act_copy_kernel (stages of 64 pixels; cps counts 32).  Fitted to 96 calls with every tile and up to eight cuts: the
// plan it picks takes 2.5 % longer than the best one measured on average, 8 % at the 90th percentile (constants fitted to half of the
// calls: 2.2 % on the other half).
static double wgrad_act_cost(int bm, int bn, int Kout, int Jdim, int split, int cps)
{
    static const double c128x128[3] = {0.568, 2.462, 1.021}, c128x64[3] = {0.371, 0.852, 0.580}, c64x128[3] = {0.424, 0.987, 0.722},
                        c64x64[3] = {0.258, 0.376, 0.420};
    const double *c = bm == 128 ? (bn == 128 ? c128x128 : c128x64) : (bn == 128 ? c64x128 : c64x64);
    const int per_cu = ceil_div((long)ceil_div(Kout, bm) * ceil_div(Jdim, bn) * split, (int)kCUs), stages = ceil_div(cps, 2);
    return std::max(per_cu * (stages * c[0] + c[1]), ceil_div(per_cu, igemm_act_occupancy(bm, bn)) * stages * c[2]) +
           (split + 1.0) * Kout * Jdim * 4.0 / 5.03e6;
}
static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
// The same for wgrad_terms_kernel, with its preparation (`elems` numbers in both tensors) and launches.  Fitted to 1,620 measured launches (45 calls, every tile,
// twelve cuts): the plan it picks takes 1.6 % longer than the best one on average.
static double wgrad_terms_cost(int bm, int bn, int Kout, int Jdim, int split, int cps, double elems)
{
    static const double c128x64[3] = {0.558, 0.684, 0.748}, c64x128[3] = {0.512, 0.882, 0.822}, c64x64[3] = {0.292, 0.371, 0.506};
    const double *c = bm == 128 ? c128x64 : bn == 128 ? c64x128 : c64x64;
    const int per_cu = ceil_div((long)ceil_div(Kout, bm) * ceil_div(Jdim, bn) * split, (int)kCUs);
    return std::max(per_cu * (cps * c[0] + c[1]), ceil_div(per_cu, wgrad_terms_occupancy(bm, bn)) * (cps * c[2] + 0.7)) +
           (split + 1.0) * Kout * Jdim * 4.0 / 5.26e6 + 11.2 + 2.05e-6 * elems;
}
constexpr double kWgradSplitLaunches = 14.7;  // what wgrad_split_cost leaves out of a call
constexpr double kWgradTermsMinFlops = 1.5e9;
static bool wgrad_may_split_terms(const rn50_conv_desc *d, long Mpix, Fp32Math math)
{
    return math == kFp32Split && !bf16_of(d) && d->c % 32 == 0 && d->k % 32 == 0 && (long)d->n * d->h * d->w * d->c < (1l << 29) && Mpix * d->k < (1l << 29);
}
struct WgradTermsRoom { size_t terms[2], total; };
static WgradTermsRoom wgrad_terms_room(const rn50_conv_desc *d, const GemmPlan &pl, int Kout, int Jdim, long Mpix)
{
    WgradTermsRoom r;
    r.terms[0] = align_up((size_t)pl.split * Kout * Jdim * sizeof(float), 256);
    r.terms[1] = r.terms[0] + align_up((size_t)d->n * d->h * d->w * d->c * 6 + kTermsZeros, 256);
    r.total = r.terms[1] + align_up((size_t)Mpix * d->k * 6 + kTermsZeros, 256);
    return r;
}

// Whether a filter gradient runs through wgrad_act_copy_kernel: bf16 activations (the fp32 image in front of them: wgrad_act_kernel)
static bool wgrad_is_copy(const rn50_conv_desc *d) { return act_of(d) == 1 && d->k % 8 == 0 && d->c % 8 == 0; }
static GemmPlan plan_wgrad_copy(const rn50_conv_desc *d, int Kout, int Jdim, long Mpix)
{
    const int pchunks = ceil_div(Mpix, kBK);
    GemmPlan best{64, 64, 1, pchunks};
    const std::shared_ptr<const Config> cfg = config();
    GemmPlan forced;
    if (forced_plan(cfg->has_wgrad_plan, cfg->wgrad_plan, &forced) || override_plan(*cfg, d, RN50_OP_BWD_WEIGHT, &forced)) {
        if (forced.split > pchunks) forced.split = pchunks;
        forced.chunks_per_split = even_stages(ceil_div(pchunks, forced.split), pchunks);
        forced.split = ceil_div(pchunks, forced.chunks_per_split);
        return forced;
    }
    double best_cost = 1e300;
    for (int bm = 128; bm >= 64; bm -= 64)
        for (int bn = 128; bn >= 64; bn -= 64) {
            if ((bm == 128 && Kout <= 64) || (bn == 128 && Jdim <= 64)) continue;
            for (int s = 1; s <= 2048; s = (s < 8 ? s + 1 : s + s / 4)) {
                if (s > 1 && pchunks / s < 2) break;
                const int cps = even_stages(ceil_div(pchunks, s), pchunks), sp = ceil_div(pchunks, cps);
                const double cost = wgrad_act_cost(bm, bn, Kout, Jdim, sp, cps);
                if (cost < best_cost) { best_cost = cost; best = GemmPlan{bm, bn, sp, cps}; }
            }
        }
    return best;
}

static GemmPlan plan_wgrad_any_tile(const rn50_conv_desc *d, int Kout, int Jdim, long Mpix, Fp32Math math)
{
    const int pchunks = ceil_div(Mpix, kBK);
    const std::shared_ptr<const Config> cfg = config();
    const bool may_split = (math == kFp32Split || math == kNoHalf) && !bf16_of(d) && d->c % 4 == 0;  // c % 4: four filter indices share a tap, one 16-byte load
    GemmPlan unit{64, 64, 1, pchunks}, best = unit;
    double unit_cost = 1e300, best_cost = 1e300;
    auto every_cut = [&](auto try_one) {
        for (int bm = 128; bm >= 64; bm -= 64)
            for (int bn = 128; bn >= 64; bn -= 64) {
                if ((bm == 128 && Kout <= 64) || (bn == 128 && Jdim <= 64)) continue;
                for (int s = 1; s <= 2048; s = (s < 8 ? s + 1 : s + s / 4)) {
                    if (s > 1 && pchunks / s < 2) break;
                    const int cps = even_stages(ceil_div(pchunks, s), pchunks);
                    try_one(bm, bn, ceil_div(pchunks, cps), cps);
                }
            }
    };
    const bool given = forced_plan(cfg->has_wgrad_plan, cfg->wgrad_plan, &unit) || override_plan(*cfg, d, RN50_OP_BWD_WEIGHT, &unit);
    if (given || tuned_plan(*cfg, d, RN50_OP_BWD_WEIGHT, &unit)) {
        if (unit.split > pchunks) unit.split = pchunks;
        unit.chunks_per_split = even_stages(ceil_div(pchunks, unit.split), pchunks);
        unit.split = ceil_div(pchunks, unit.chunks_per_split);
        if (given) {
            unit.products = may_split && wgrad_split_as_precise(Mpix, unit.split, unit.split);
            return unit;
        }
    } else {
        every_cut([&](int bm, int bn, int sp, int cps) {
            const int occ = wgrad_occupancy(bm, bn);
            const double chunk_clks = 4096.0 * (bm * bn / 16384.0);
            const int per_cu = ceil_div((long)ceil_div(Kout, bm) * ceil_div(Jdim, bn) * sp, (int)kCUs);        // workgroups the busiest CU runs
            const double conc = std::min(occ, per_cu);                                                // of which this many at a time
            // a stage costs its MFMA time, but no less than what the load latency allows at this concurrency
            const double stage = std::max(chunk_clks, 3000.0 / conc);
            const double cost = per_cu * (cps + 3.0) * stage + kLaunchClks + (sp + 1.0) * Kout * Jdim * 4.0 / kBytesPerClk;
            if (cost < unit_cost) { unit_cost = cost; unit = GemmPlan{bm, bn, sp, cps}; }
        });
    }
    if (may_split && wgrad_split_as_precise(Mpix, unit.split, pchunks))  // in some number of ranges
        every_cut([&](int bm, int bn, int sp, int cps) {
            if (!wgrad_split_as_precise(Mpix, unit.split, sp)) return;
            const double cost = wgrad_split_cost(bm, bn, Kout, Jdim, sp, cps);
            if (cost < best_cost) { best_cost = cost; best = GemmPlan{bm, bn, sp, cps, true}; }
        });
    if (wgrad_may_split_terms(d, Mpix, math)) {
        for (const PlanRow &t : cfg->operand_plans)
            if (plan_matches(t, d, RN50_OP_BWD_WEIGHT) && (t.bm == 64 || t.bn == 64)) {
                const int cps = ceil_div(pchunks, std::min(t.split, pchunks));
                return GemmPlan{t.bm, t.bn, ceil_div(pchunks, cps), cps, true, true};
            }
    }
    if (best.products && 2.0 * Mpix * Kout * Jdim >= kWgradTermsMinFlops && wgrad_may_split_terms(d, Mpix, math)) {
        // both tensors split beforehand: the same products in no fewer ranges, so no larger an error
        const double elems = (double)d->n * d->h * d->w * d->c + (double)Mpix * d->k;
        const int ranges = best.split;
        best_cost = 0.97 * (best_cost + kWgradSplitLaunches);
        every_cut([&](int bm, int bn, int sp, int cps) {
            if ((bm == 128 && bn == 128) || sp < ranges) return;
            const double cost = wgrad_terms_cost(bm, bn, Kout, Jdim, sp, cps, elems);
            if (cost < best_cost) { best_cost = cost; best = GemmPlan{bm, bn, sp, cps, true, true}; }
        });
    }
    return best.products ? best : unit;
}

template <int MODE, int PREC, bool INAFF, int ACT, bool STATS, int BK>
static void launch_igemm_bk(const IgemmPlan &pl, const IgemmP &p, hipStream_t st)
{
    const dim3 grid(pl.grid), block(kConvThreads);
    if (pl.bm == 128 && pl.bn == 128) hipLaunchKernelGGL((igemm_kernel<128, 128, MODE, PREC, INAFF, ACT, STATS, BK>), grid, block, 0, st, p);
    else if (pl.bm == 128) hipLaunchKernelGGL((igemm_kernel<128, 64, MODE, PREC, INAFF, ACT, STATS, BK>), grid, block, 0, st, p);
    else if (pl.bn == 128) hipLaunchKernelGGL((igemm_kernel<64, 128, MODE, PREC, INAFF, ACT, STATS, BK>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((igemm_kernel<64, 64, MODE, PREC, INAFF, ACT, STATS, BK>), grid, block, 0, st, p);
}

// p.kchunks counts stages of igemm_bk() elements: the instantiation with that stage length
template <int MODE, int PREC, bool INAFF = false, int ACT = 0, bool STATS = false>
static void launch_igemm_mode(const IgemmPlan &pl, const IgemmP &p, hipStream_t st)
{
    if constexpr (PREC == 1 && MODE <= 1) {
        if (igemm_bk(true, ACT, p.Cin) == 2 * kBK) {
            launch_igemm_bk<MODE, PREC, INAFF, ACT, STATS, 2 * kBK>(pl, p, st);
            return;
        }
    }
    launch_igemm_bk<MODE, PREC, INAFF, ACT, STATS, kBK>(pl, p, st);
}

// A launch with fp32 operands: on the fp32 instruction or with split operands
#define RN50_FP32(MODE_, ...) \
    do { if (split) launch_igemm_mode<MODE_, 2, __VA_ARGS__>(pl, p, st); else launch_igemm_mode<MODE_, 0, __VA_ARGS__>(pl, p, st); } while (0)

// The forward launches that also gather the output's statistics (p.stat_mean set): no dilation, so the vector gather
// (MODE 0) or the scalar one (MODE 2).
static void launch_igemm_stats(const IgemmPlan &pl, const IgemmP &p, bool bf16, bool split, int act, hipStream_t st)
{
    const bool fast = p.Cin % kBK == 0 && act != 2;
    if (act == 1) {
        if (p.in_scale) launch_igemm_mode<0, 1, true, 1, true>(pl, p, st);
        else if (fast) launch_igemm_mode<0, 1, false, 1, true>(pl, p, st);
        else launch_igemm_mode<2, 1, false, 1, true>(pl, p, st);
    } else if (act == 2) {
        launch_igemm_mode<2, 1, false, 2, true>(pl, p, st);
    } else if (p.in_scale) {
        if (bf16) launch_igemm_mode<0, 1, true, 0, true>(pl, p, st);
        else RN50_FP32(0, true, 0, true);
    } else if (bf16) {
        if (fast) launch_igemm_mode<0, 1, false, 0, true>(pl, p, st);
        else launch_igemm_mode<2, 1, false, 0, true>(pl, p, st);
    } else {
        if (fast) RN50_FP32(0, false, 0, true);
        else RN50_FP32(2, false, 0, true);
    }
}

template <bool O16, bool APPLY = false>
static void launch_tail_reduce(const IgemmPlan &pl, const IgemmP &p, hipStream_t st, const TailApply &ap = TailApply{})
{
    const dim3 grid(ceil_div(pl.bm * pl.bn / 4, 256), pl.tail_tiles), block(256);
    if (pl.bm == 128 && pl.bn == 128) hipLaunchKernelGGL((igemm_tail_reduce_kernel<128, 128, O16, APPLY>), grid, block, 0, st, p, ap);
    else if (pl.bm == 128) hipLaunchKernelGGL((igemm_tail_reduce_kernel<128, 64, O16, APPLY>), grid, block, 0, st, p, ap);
    else if (pl.bn == 128) hipLaunchKernelGGL((igemm_tail_reduce_kernel<64, 128, O16, APPLY>), grid, block, 0, st, p, ap);
    else hipLaunchKernelGGL((igemm_tail_reduce_kernel<64, 64, O16, APPLY>), grid, block, 0, st, p, ap);
}

template <bool O16>
static void launch_tail_reduce_stats(const IgemmPlan &pl, const IgemmP &p, hipStream_t st)
{
    const dim3 grid(pl.bn / 32, pl.tail_tiles), block(256);
    if (pl.bm == 128 && pl.bn == 128) hipLaunchKernelGGL((igemm_tail_reduce_stats_kernel<128, 128, O16>), grid, block, 0, st, p);
    else if (pl.bm == 128) hipLaunchKernelGGL((igemm_tail_reduce_stats_kernel<128, 64, O16>), grid, block, 0, st, p);
    else if (pl.bn == 128) hipLaunchKernelGGL((igemm_tail_reduce_stats_kernel<64, 128, O16>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((igemm_tail_reduce_stats_kernel<64, 64, O16>), grid, block, 0, st, p);
}

// Runs out[M][Nout] (+ optional stride-2 scatter) and, when tail tiles are split, the ordered sum of their pieces.
// act: storage of the gathered operand and of the output (see act_of).
// ap (a forward pass, fp32 output): what to make of the output besides; returns whether it was made (where every tile is split the
// ordered sum makes it, a launch and a pass less), else it is the caller's to do.
static bool run_igemm(IgemmWideP p, const IgemmPlan &pl, float *out, float *partials, bool bf16, int act, hipStream_t st,
                      const TailApply *ap = nullptr)
{
    const bool fast = p.Cin % kBK == 0 && act != 2;  // an fp32 input beside bf16 activations goes through the scalar gather
    const bool split = pl.products;
    p.kchunks = ceil_div(p.Kdim, fast ? igemm_bk(bf16, act, p.Cin) : kBK);
    p.tiles_m = ceil_div(p.M, pl.bm);
    p.tiles_n = ceil_div(p.Nout, pl.bn);
    p.full_items = pl.full_items;
    p.tail_tiles = pl.tail_tiles;
    p.tail_split = pl.tail_split;
    p.tail_chunks = pl.tail_chunks;
    p.out = out;
    p.partial = partials;
    p.div_ohw = make_fastdiv(p.OH * p.OW);
    p.div_ow = make_fastdiv(p.OW);
    p.div_cin = make_fastdiv(p.Cin);
    p.div_s = make_fastdiv(p.S);
    p.div_rs = make_fastdiv(p.R * p.S);
    if (pl.kind == kSmall) {
        launch_igemm_small(pl.bm, pl.bn, pl.grid, p, st);
        return false;
    }
    if (pl.kind == kHalf) {
        launch_igemm_half(pl.bm, pl.bn, pl.grid, p, st);
    } else if (pl.kind == kPre) {
        launch_igemm_pre(pl.bm, pl.bn, pl.grid, p, st);
    } else if (pl.kind == kAct) {
        launch_igemm_act(pl.bm, pl.bn, pl.grid, p, st);
    } else if (p.stat_mean) {
        launch_igemm_stats(pl, p, bf16, split, act, st);  // callers have checked: a forward pass (sd == 1)
    } else if (act == 1) {
        if (p.in_scale) launch_igemm_mode<0, 1, true, 1>(pl, p, st);
        else if (fast && p.sd == 1) launch_igemm_mode<0, 1, false, 1>(pl, p, st);
        else if (fast) launch_igemm_mode<1, 1, false, 1>(pl, p, st);
        else launch_igemm_mode<2, 1, false, 1>(pl, p, st);
    } else if (act == 2) {
        launch_igemm_mode<2, 1, false, 2>(pl, p, st);
    } else if (p.in_scale) {  // callers have checked: Cin % 32 == 0 and no dilation
        if (bf16) launch_igemm_mode<0, 1, true>(pl, p, st);
        else RN50_FP32(0, true);
    } else if (bf16) {
        if (fast && p.sd == 1) launch_igemm_mode<0, 1>(pl, p, st);
        else if (fast) launch_igemm_mode<1, 1>(pl, p, st);
        else launch_igemm_mode<2, 1>(pl, p, st);
    } else {
        if (fast && p.sd == 1) RN50_FP32(0, false);
        else if (fast) RN50_FP32(1, false);
        else RN50_FP32(2, false);
    }
    if (pl.tail_split > 1) {
        if (p.stat_mean) {
            if (act) launch_tail_reduce_stats<true>(pl, p, st);
            else launch_tail_reduce_stats<false>(pl, p, st);
        } else {
            if (act) launch_tail_reduce<true>(pl, p, st);
            else if (ap && !pl.full_items && !p.scatter2 && p.Nout % 4 == 0) {
                launch_tail_reduce<false, true>(pl, p, st, *ap);
                return true;
            } else launch_tail_reduce<false>(pl, p, st);
        }
    }
    return false;
}

// Workspace of a forward or data-gradient call: [partial tiles][prepared filter], the latter only where the plan's kernel takes one.
static size_t igemm_part_bytes(const IgemmPlan &pl) { return pl.kind == kGeneral ? pl.ws_floats * sizeof(float) : align_up(pl.ws_floats * sizeof(float), 256); }
// The prepared filter of a call: the one it was given, or prepared now in the workspace behind the partial tiles.  Operands as fp16 halves:
// both prepared there, the gathered tensor of `pixels` pixels among them.
static void set_planes(IgemmWideP &p, const IgemmPlan &pl, const char *planes, long pixels, void *ws, hipStream_t st)
{
    if (pl.kind == kGeneral || pl.kind == kSmall) return;
    p.plane_rows = plane_rows_of(p.Nout);
    p.planes = planes;
    if (planes && pl.kind != kHalf) return;  // a filter given as bf16 terms is none of this call's: options set since a context was made can plan halves
    char *own = (char *)ws + igemm_part_bytes(pl);
    p.planes = own;
    if (pl.kind != kHalf) {
        launch_filter_planes(p.Nout, p.Kdim, pl.kind == kAct, p.b, own, st);
        return;
    }
    const HalfRoom room = half_room(pixels, p.Cin, p.Nout, p.Kdim);
    unsigned *marks = (unsigned *)(own + room.marks);
    p.planes = own + room.planes;
    p.halves = own + room.halves;
    p.half_up = (const int *)own;
    p.half_any = marks;
    p.half_marks[0] = marks + 1;
    p.half_marks[1] = marks + room.nmarks - p.Nout;
    HalfPrep q{};
    q.in_scale = p.in_scale;
    q.in_shift = p.in_shift;
    q.div_c4 = make_fastdiv(p.Cin / 4);
    q.marks = marks;
    q.nmarks = room.nmarks;
    for (int i = 0; i < 2; ++i) {
        HalfOperand &o = q.op[i];
        o.src = i ? p.b : p.a;
        o.dst = own + (i ? room.planes : room.halves);
        const long count = i ? (long)p.Nout * p.Kdim : pixels * p.Cin;
        o.n4 = (unsigned)(count / 4);
        o.n8 = (unsigned)(i ? (long)p.plane_rows * p.Kdim / 8 : count / 8);
        o.kind = i ? (p.flip_taps ? kHalfFlipped : kHalfFilter) : kHalfPixels;
        o.blocks = std::min(kHalfShares, ceil_div(o.n4, 1024));
        o.split_blocks = std::min(2048, ceil_div(o.n8, 512));
        o.rows = p.Nout;
        o.plane_rows = p.plane_rows;
        o.kdim = p.Kdim;
        o.taps = p.R * p.S;
        o.div8 = make_fastdiv(!i ? p.Cin / 8 : p.flip_taps ? p.plane_rows : p.Kdim / 8);
        o.div_k = make_fastdiv(p.Cin);
        o.part = (unsigned *)(own + room.part) + i * kHalfShares;
        o.marks = const_cast<unsigned *>(p.half_marks[i]);
        o.any = marks;
        o.up = (int *)own + i;
    }
    launch_half_prep(q, st);
}

struct BwdDataPlan { IgemmPlan g; bool scatter; size_t wt_bytes, part_bytes; };  // part_bytes: partial tiles and prepared filter
static BwdDataPlan plan_bwd_data(const rn50_conv_desc *d, Fp32Math math, bool given = false)
{
    const Geom ge = geom(d);
    BwdDataPlan b;
    b.scatter = is_scatter2(d);
    const long M = b.scatter ? ge.Mout : ge.Min;
    const int Kd = d->r * d->s * d->k;
    b.g = plan_igemm(d, RN50_OP_BWD_DATA, M, d->c, Kd, true, d->k, math, given);
    b.wt_bytes = align_up((size_t)d->k * d->r * d->s * d->c * sizeof(float), 256);
    b.part_bytes = igemm_part_bytes(b.g) + b.g.prep_bytes;
    return b;
}

// Whether the first layer's output is a whole number of its kernels' tiles
static bool stem_whole(const Geom &ge) { return ge.P % kStemTH == 0 && ge.Q % kStemTW == 0; }
// Whether its forward kernel leaves the batch statistics of its tiles (not on the fp32 instruction)
static bool stem_stats(const rn50_conv_desc *d, const Geom &ge, Fp32Math math)
{
    return stem_layer(d) && stem_whole(ge) && (act_of(d) || math == kFp32Split || math == kNoHalf);
}

// Forward pass that also gathers the output's batch statistics: workspace = [the forward pass's own][statistics region].
// The region holds mean and squared deviations per (row tile, output channel), or, for a shape whose forward pass does not
// run through the tiled kernel, the band partials of the separate statistics pass; it is sized for both.
struct FwdStatsPlan { IgemmPlan g; int tiles_m, rows; size_t conv_bytes, stat_bytes; };
static size_t stat_room(const rn50_conv_desc *d, const Geom &ge, int rows)
{
    return align_up(std::max((size_t)2 * ceil_div(ge.Mout, rows) * d->k * sizeof(float), rn50_bn_workspace_bytes(d->n, d->k, ge.P, ge.Q)), 256);
}
// plan_small for a call whose plan is pl.  Forward pass: with and without statistics the same kernel.
static IgemmPlan small_fwd(const rn50_conv_desc *d, const Geom &ge, const IgemmPlan &pl)
{
    return plan_small(d, RN50_OP_FWD, ge.Mout, d->k, ge.Kdim, d->c, pl, 0.0, d->k % 4 ? 0 : stat_room(d, ge, pl.bm));
}
static IgemmPlan small_bwd(const rn50_conv_desc *d, const BwdDataPlan &b, bool flipped)
{
    const Geom ge = geom(d);
    return plan_small(d, RN50_OP_BWD_DATA, b.scatter ? ge.Mout : ge.Min, d->c, d->r * d->s * d->k, d->k, b.g, flipped ? 0.0 : kFlipLaunch);
}
static FwdStatsPlan plan_fwd_stats(const rn50_conv_desc *d, Fp32Math math, bool given = false)
{
    const Geom ge = geom(d);
    FwdStatsPlan f;
    f.g = plan_igemm(d, RN50_OP_FWD, ge.Mout, d->k, ge.Kdim, true, d->c, math, given);
    f.rows = stem_stats(d, ge, math) ? kStemTH * kStemTW : f.g.bm;
    f.tiles_m = ceil_div(ge.Mout, f.rows);
    f.conv_bytes = align_up(igemm_part_bytes(f.g) + f.g.prep_bytes, 256);
    f.stat_bytes = stat_room(d, ge, f.rows);
    if (math == kFp32Split || math == kNoHalf) {
        const IgemmPlan sm = small_fwd(d, ge, f.g);
        if (sm.grid) {
            f.rows = sm.bm;
            f.tiles_m = ceil_div(ge.Mout, f.rows);
            f.stat_bytes = std::max(f.stat_bytes, stat_room(d, ge, f.rows));
        }
    }
    return f;
}

}  // namespace rn50

using namespace rn50;

// Workgroups of the first layer's own filter-gradient kernel (0: the layer goes through the general kernel).
static int stem_wgrad_grid(const rn50_conv_desc *d, const Geom &ge)
{
    // with bf16 activations whole tiles only: pixels outside the output multiply image values with zeros, which an infinite value shows
    if (!stem_layer(d) || (act_of(d) && !stem_whole(ge))) return 0;
    const int ntiles = d->n * ceil_div(ge.P, kStemTH) * ceil_div(ge.Q, kStemTW);
    return std::min(ntiles, 2 * (int)kCUs);
}

extern "C" size_t rn50_conv_workspace_bytes(const rn50_conv_desc *d, int op)
{
    const ConfigScope snapshot;
    if (conv_check("rn50_conv_workspace_bytes", d) != RN50_OK) return 0;
    return conv_workspace(d, op, kFp32Split, false);
}

static size_t wgrad_bytes(const rn50_conv_desc *d, const GemmPlan &pl, const Geom &ge)
{
    return pl.terms ? wgrad_terms_room(d, pl, d->k, ge.Kdim, ge.Mout).total : (size_t)pl.split * d->k * ge.Kdim * sizeof(float);
}

size_t rn50::conv_workspace(const rn50_conv_desc *d, int op, Fp32Math math, bool given)
{
    const ConfigScope snapshot;
    const Geom ge = geom(d);
    if (op == RN50_OP_FWD) {
        const IgemmPlan pl = plan_igemm(d, RN50_OP_FWD, ge.Mout, d->k, ge.Kdim, true, d->c, math, given);
        return igemm_part_bytes(pl) + pl.prep_bytes;
    }
    if (op == RN50_OP_BWD_DATA) {
        const BwdDataPlan b = plan_bwd_data(d, math, given);
        return b.wt_bytes + b.part_bytes;
    }
    if (op == RN50_OP_BWD_WEIGHT) {
        if (stem_wgrad_grid(d, ge)) return (size_t)stem_wgrad_grid(d, ge) * d->k * ge.Kdim * sizeof(float);
        const GemmPlan pl = wgrad_is_copy(d) ? plan_wgrad_copy(d, d->k, ge.Kdim, ge.Mout) : plan_wgrad(d, d->k, ge.Kdim, ge.Mout, math);
        return wgrad_bytes(d, pl, ge);
    }
    if (op == RN50_OP_BWD_DATA_FLIPPED) return plan_bwd_data(d, math, given).part_bytes;
    if (op == RN50_OP_FWD_BNSTATS) {
        const FwdStatsPlan f = plan_fwd_stats(d, math, given);
        return f.conv_bytes + f.stat_bytes;
    }
    return 0;
}

extern "C" int rn50_conv_plan(const rn50_conv_desc *d, int op, int *bm, int *bn, int *split, int *workgroups)
{
    const ConfigScope snapshot;
    if (int rc = conv_check("rn50_conv_plan", d)) return rc;
    const Geom ge = geom(d);
    int v[4];
    if (op == RN50_OP_FWD || op == RN50_OP_FWD_BNSTATS || op == RN50_OP_BWD_DATA || op == RN50_OP_BWD_DATA_FLIPPED) {
        const bool fwd = op == RN50_OP_FWD || op == RN50_OP_FWD_BNSTATS;
        const BwdDataPlan b = fwd ? BwdDataPlan{} : plan_bwd_data(d, kFp32Split);
        IgemmPlan pl = fwd ? plan_igemm(d, RN50_OP_FWD, ge.Mout, d->k, ge.Kdim, true, d->c, kFp32Split, false) : b.g;
        const IgemmPlan sm = fwd ? small_fwd(d, ge, pl) : small_bwd(d, b, op == RN50_OP_BWD_DATA_FLIPPED);
        if (sm.grid) pl = sm;
        v[0] = pl.bm; v[1] = pl.bn; v[2] = pl.tail_tiles ? pl.tail_split : 1; v[3] = pl.grid;
        if (fwd && stem_layer(d) && (op == RN50_OP_FWD || !act_of(d) || stem_whole(ge))) {
            // the first layer's own forward kernel (same shapes as its filter-gradient kernel): tiles of 8 x 16 pixels x 64 filters
            v[0] = kStemTH * kStemTW; v[1] = 64; v[2] = 1;
            v[3] = std::min(d->n * ceil_div(ge.P, kStemTH) * ceil_div(ge.Q, kStemTW), (act_of(d) ? 3 : 2) * (int)kCUs);
        }
    } else if (op == RN50_OP_BWD_WEIGHT) {
        const GemmPlan pl = wgrad_is_copy(d) ? plan_wgrad_copy(d, d->k, ge.Kdim, ge.Mout) : plan_wgrad(d, d->k, ge.Kdim, ge.Mout, kFp32Split);
        v[0] = pl.bm; v[1] = pl.bn; v[2] = pl.split; v[3] = ceil_div(d->k, pl.bm) * ceil_div(ge.Kdim, pl.bn) * pl.split;
        if (const int sgrid = stem_wgrad_grid(d, ge)) {  // the first layer's own kernel: 64 filters x 160 filter elements, one partial per workgroup
            v[0] = 64; v[1] = 160; v[2] = sgrid; v[3] = sgrid;
        }
    } else {
        return fail(RN50_EINVAL, "rn50_conv_plan: unknown operation %d", op);
    }
    if (bm) *bm = v[0];
    if (bn) *bn = v[1];
    if (split) *split = v[2];
    if (workgroups) *workgroups = v[3];
    return RN50_OK;
}

// stats (may be null): [2][row tiles][K] floats for the output's per-tile statistics; *gathered tells whether they were left
static int conv_fwd_impl(const char *who, const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift,
                         const float *w, float *y, void *ws, size_t ws_bytes, void *stream, float *stats = nullptr, bool *gathered = nullptr,
                         Fp32Math math = kFp32Split, const char *planes = nullptr, const TailApply *ap = nullptr, int stat_rows = 0);

extern "C" int conv2d_fwd(const rn50_conv_desc *d, const float *x, const float *w, float *y, void *ws, size_t ws_bytes,
                          void *stream)
{
    return conv_fwd_impl("conv2d_fwd", d, x, nullptr, nullptr, w, y, ws, ws_bytes, stream);
}

extern "C" int conv2d_fwd_bnrelu_input(const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift,
                                       const float *w, float *y, void *ws, size_t ws_bytes, void *stream)
{
    RN50_REQUIRE(in_scale && in_shift && aligned16(in_scale) && aligned16(in_shift), RN50_EINVAL,
                 "conv2d_fwd_bnrelu_input: scale and shift must be non-null and 16-byte aligned");
    RN50_REQUIRE(d && d->c % kBK == 0, RN50_EUNSUPPORTED, "conv2d_fwd_bnrelu_input: the channel count must be a multiple of 32");
    return conv_fwd_impl("conv2d_fwd_bnrelu_input", d, x, in_scale, in_shift, w, y, ws, ws_bytes, stream);
}

static int conv_fwd_impl(const char *who, const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift,
                         const float *w, float *y, void *ws, size_t ws_bytes, void *stream, float *stats, bool *gathered, Fp32Math math,
                         const char *planes, const TailApply *ap, int stat_rows)
{
    const ConfigScope snapshot;
    if (gathered) *gathered = false;
    if (int rc = conv_check(who, d)) return rc;
    RN50_REQUIRE(x && w && y, RN50_EINVAL, "%s: null pointer", who);
    RN50_REQUIRE(aligned16(x) && aligned16(w) && aligned16(y) && aligned16(ws), RN50_EINVAL, "%s: pointers must be 16-byte aligned", who);
    const Geom ge = geom(d);
    if (in_scale && act_of(d)) math = kNoPlanes;  // the copies of igemm_act_kernel apply no transform: the general kernel
    IgemmPlan pl = plan_igemm(d, RN50_OP_FWD, ge.Mout, d->k, ge.Kdim, true, d->c, math, planes != nullptr);
    size_t need = igemm_part_bytes(pl) + pl.prep_bytes;
    while (math != kNoPlanes && need && (ws_bytes < need || !ws)) {  // less room than the query names: see less_room
        math = less_room(math);
        pl = plan_igemm(d, RN50_OP_FWD, ge.Mout, d->k, ge.Kdim, true, d->c, math, false);
        need = igemm_part_bytes(pl) + pl.prep_bytes;
    }
    RN50_REQUIRE(ws_bytes >= need && (need == 0 || ws), RN50_EWORKSPACE, "%s: workspace too small (%zu < %zu)", who, ws_bytes, need);
    RN50_REQUIRE(!in_scale || act_of(d) != 2, RN50_EUNSUPPORTED, "%s: the fused input transform needs a bf16 or fp32 input of the variant's own type", who);
    // (evaluation, ap, as the training forward of its context: the same sums, and so the same logits from a training batch's own statistics; with other
    // sums those differ by 1.2e-5 for one to three images, whose 49 to 147 pixels in the last stage leave statistics that magnify roundings)
    if (math == kFp32Split || math == kNoHalf) {
        const IgemmPlan sm = small_fwd(d, ge, pl);
        if (sm.grid && (!stats || stat_rows == sm.bm)) pl = sm;
    }
    const bool swhole = stem_stats(d, ge, math);
    if (stem_layer(d) && !in_scale && !(act_of(d) && stats && !swhole)) {
        // the network's first layer has kernels of its own (input tile and filter in LDS)
        const int tiles_h = ceil_div(ge.P, kStemTH), tiles_w = ceil_div(ge.Q, kStemTW), ntiles = d->n * tiles_h * tiles_w;
        if (act_of(d) || math == kFp32Split || math == kNoHalf) {
            StemMP sp{};
            sp.x = x; sp.w = w; sp.y = y;
            sp.N = d->n; sp.IH = d->h; sp.IW = d->w; sp.OH = ge.P; sp.OW = ge.Q;
            sp.tiles_h = tiles_h; sp.tiles_w = tiles_w; sp.ntiles = ntiles;
            if (stats && swhole) {
                sp.mean = stats;
                sp.m2 = stats + (size_t)ntiles * d->k;
                *gathered = true;
            }
            launch_stem_fwd(act_of(d) ? 1 : 2, sp.mean != nullptr, sp, (hipStream_t)stream);
        } else {
            StemP sp{};
            sp.x = x; sp.w = w; sp.y = y;
            sp.N = d->n; sp.IH = d->h; sp.IW = d->w; sp.OH = ge.P; sp.OW = ge.Q;
            sp.tiles_h = tiles_h; sp.tiles_w = tiles_w; sp.ntiles = ntiles;
            hipLaunchKernelGGL(stem_fwd_kernel, dim3(std::min(sp.ntiles, 3 * (int)kCUs)), dim3(kConvThreads), 0, (hipStream_t)stream, sp);
        }
        if (ap)
            if (int rc = bn_fwd_apply(d->n, d->k, ge.P, ge.Q, RN50_LAYOUT_NHWC, y, ap->scale, ap->shift, ap->residual, ap->relu, ap->z, nullptr, stream)) return rc;
        return launch_status(who);
    }
    IgemmWideP p{};
    p.a = x; p.b = w; p.in_scale = in_scale; p.in_shift = in_shift;
    p.IH = d->h; p.IW = d->w; p.Cin = d->c; p.OH = ge.P; p.OW = ge.Q; p.Nout = d->k; p.R = d->r; p.S = d->s;
    p.so = d->stride; p.off = -d->pad; p.sd = 1; p.M = (int)ge.Mout; p.Kdim = ge.Kdim; p.scatter2 = 0;
    if (stats) {
        p.stat_mean = stats;
        p.stat_m2 = stats + (size_t)ceil_div(ge.Mout, pl.bm) * d->k;
        if (gathered) *gathered = true;
    }
    set_planes(p, pl, planes, ge.Min, ws, (hipStream_t)stream);
    if (!run_igemm(p, pl, y, (float *)ws, bf16_of(d), act_of(d), (hipStream_t)stream, ap) && ap)
        if (int rc = bn_fwd_apply(d->n, d->k, ge.P, ge.Q, RN50_LAYOUT_NHWC, y, ap->scale, ap->shift, ap->residual, ap->relu, ap->z, nullptr, stream)) return rc;
    return launch_status(who);
}

extern "C" int conv2d_fwd_bnstats(const rn50_conv_desc *d, const float *x, const float *in_scale_or_null, const float *in_shift_or_null,
                                  const float *w, float *y, const float *gamma, const float *beta, float eps, float *save_mean,
                                  float *save_invstd, float *scale, float *shift, void *ws, size_t ws_bytes, void *stream)
{
    return conv_fwd_bnstats_math(kFp32Split, d, x, in_scale_or_null, in_shift_or_null, w, nullptr, y, gamma, beta, eps, save_mean, save_invstd, scale, shift, ws,
                                   ws_bytes, (hipStream_t)stream);
}

int rn50::conv_fwd_math(Fp32Math math, const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift, const float *w, const char *planes,
                          float *y, void *ws, size_t ws_bytes, hipStream_t st)
{
    return conv_fwd_impl("conv2d_fwd", d, x, in_scale, in_shift, w, y, ws, ws_bytes, st, nullptr, nullptr, math, planes);
}

int rn50::conv_fwd_apply_math(Fp32Math math, const rn50_conv_desc *d, const float *x, const float *w, const char *planes, float *y, const float *scale,
                              const float *shift, const float *residual, int relu, float *z, void *ws, size_t ws_bytes, hipStream_t st)
{
    const TailApply ap{scale, shift, residual, z, relu};
    return conv_fwd_impl("conv2d_fwd", d, x, nullptr, nullptr, w, y, ws, ws_bytes, st, nullptr, nullptr, math, planes, &ap);
}

size_t rn50::conv_planes_bytes(const rn50_conv_desc *d, int op)
{
    const ConfigScope snapshot;
    const Geom ge = geom(d);
    const bool fwd = op == RN50_OP_FWD;
    const IgemmPlan pl = fwd ? plan_igemm(d, op, ge.Mout, d->k, ge.Kdim, true, d->c, kFp32Split, true) : plan_bwd_data(d, kFp32Split, true).g;
    return pl.kind == kPre || pl.kind == kAct ? filter_planes_bytes(fwd ? d->k : d->c, fwd ? ge.Kdim : d->r * d->s * d->k, pl.kind == kAct) : 0;
}

int rn50::conv_fwd_bnstats_math(Fp32Math math, const rn50_conv_desc *d, const float *x, const float *in_scale_or_null, const float *in_shift_or_null,
                                  const float *w, const char *planes, float *y, const float *gamma, const float *beta, float eps, float *save_mean,
                                  float *save_invstd, float *scale, float *shift, void *ws, size_t ws_bytes, hipStream_t stream)
{
    const ConfigScope snapshot;
    const char *who = "conv2d_fwd_bnstats";
    if (int rc = conv_check(who, d)) return rc;
    RN50_REQUIRE(gamma && beta && save_mean && save_invstd && scale && shift, RN50_EINVAL, "%s: null pointer", who);
    RN50_REQUIRE(aligned16(gamma) && aligned16(beta) && aligned16(save_mean) && aligned16(save_invstd) && aligned16(scale) && aligned16(shift),
                 RN50_EINVAL, "%s: pointers must be 16-byte aligned", who);
    RN50_REQUIRE((in_scale_or_null == nullptr) == (in_shift_or_null == nullptr), RN50_EINVAL, "%s: scale and shift of the input go together", who);
    RN50_REQUIRE(aligned16(in_scale_or_null) && aligned16(in_shift_or_null), RN50_EINVAL, "%s: pointers must be 16-byte aligned", who);
    RN50_REQUIRE(!in_scale_or_null || d->c % kBK == 0, RN50_EUNSUPPORTED, "%s: with a fused input transform the channel count must be a multiple of 32", who);
    RN50_REQUIRE(d->k % 4 == 0, RN50_EUNSUPPORTED, "%s: K must be a multiple of 4", who);
    RN50_REQUIRE(eps >= 0.f, RN50_EINVAL, "%s: negative eps", who);
    const Geom ge = geom(d);
    if (in_scale_or_null && act_of(d)) math = kNoPlanes;  // see conv_fwd_impl
    FwdStatsPlan f = plan_fwd_stats(d, math, planes != nullptr);
    while (math != kNoPlanes && ws_bytes < f.conv_bytes + f.stat_bytes) {  // less room than the query names
        math = less_room(math);
        f = plan_fwd_stats(d, math);
    }
    RN50_REQUIRE(ws && aligned16(ws) && ws_bytes >= f.conv_bytes + f.stat_bytes, RN50_EWORKSPACE, "%s: workspace too small (%zu < %zu)", who,
                 ws_bytes, f.conv_bytes + f.stat_bytes);
    float *stats = (float *)((char *)ws + f.conv_bytes);
    bool gathered = false;
    if (int rc = conv_fwd_impl(who, d, x, in_scale_or_null, in_shift_or_null, w, y, ws, f.conv_bytes, stream, stats, &gathered, math, planes, nullptr, f.rows)) return rc;
    if (gathered) {
        // (the forward pass of a training context keeps its order of sums)
        bn_finalize_partials(act_of(d) || math != kFp32Unit, ge.Mout, d->k, f.tiles_m, f.rows, stats, stats + (size_t)f.tiles_m * d->k, gamma, beta, eps,
                             save_mean, save_invstd, scale, shift, (hipStream_t)stream);
        return launch_status(who);
    }
    // no tiled kernel ran: the separate pass over y
    if (act_of(d))
        return bn_stats_scale_shift_bf16(d->n, d->k, ge.P, ge.Q, RN50_LAYOUT_NHWC, (const uint16_t *)y, gamma, beta, eps, save_mean, save_invstd,
                                         scale, shift, stats, f.stat_bytes, stream);
    return bn_stats_scale_shift(d->n, d->k, ge.P, ge.Q, RN50_LAYOUT_NHWC, y, gamma, beta, eps, save_mean, save_invstd, scale, shift, stats,
                                f.stat_bytes, stream);
}

// Data gradient with the filter already flipped and transposed (wt[c][R-1-r][S-1-s][k] = w[k][r][s][c]): a
// forward-type gather over dy.  ws = the implicit GEMM's partial tiles only.
int rn50::conv_bwd_data_pretransposed(Fp32Math math, const rn50_conv_desc *d, const float *dy, const float *wt, float *dx, void *ws,
                                      size_t ws_bytes, hipStream_t st, const char *planes, bool flipped)
{
    const ConfigScope snapshot;
    const Geom ge = geom(d);
    BwdDataPlan b = plan_bwd_data(d, math, planes != nullptr);
    while (math != kNoPlanes && b.part_bytes && (ws_bytes < b.part_bytes || !ws)) b = plan_bwd_data(d, math = less_room(math));  // less room than the query names
    RN50_REQUIRE(act_of(d) != 2, RN50_EUNSUPPORTED, "conv2d_bwd_data: RN50_DTYPE_BF16_ACT_F32IN is for the forward pass and the filter gradient");
    RN50_REQUIRE(ws_bytes >= b.part_bytes && (b.part_bytes == 0 || ws), RN50_EWORKSPACE,
                 "conv2d_bwd_data: workspace too small (%zu < %zu)", ws_bytes, b.part_bytes);
    IgemmWideP p{};
    p.a = dy; p.b = wt;
    p.IH = ge.P; p.IW = ge.Q; p.Cin = d->k; p.Nout = d->c; p.R = d->r; p.S = d->s;
    p.Kdim = d->r * d->s * d->k;
    if (b.scatter) {
        // dx[n,2p,2q,:] = dy[n,p,q,:] * W, the other three pixels of each 2x2 cell receive no tap
        p.OH = ge.P; p.OW = ge.Q; p.so = 1; p.off = 0; p.sd = 1; p.M = (int)ge.Mout; p.scatter2 = 1;
    } else {
        p.OH = d->h; p.OW = d->w; p.so = 1; p.off = d->pad - (d->r - 1); p.sd = d->stride; p.M = (int)ge.Min; p.scatter2 = 0;
        if (d->stride == 2 && d->h % 2 == 0 && d->w % 2 == 0 && d->k % kBK == 0) {
            // rows grouped by the parity class of their pixel: a tile inside one class skips the taps that never reach it
            p.OH = d->h / 2; p.OW = d->w / 2; p.scatter2 = 2;
            p.div_class = make_fastdiv(p.M / 4);
        }
    }
    if (math == kFp32Split || math == kNoHalf) {
        const IgemmPlan sm = small_bwd(d, b, flipped);
        if (sm.grid) b.g = sm;
    }
    p.flip_taps = (b.g.kind == kHalf || b.g.kind == kSmall) && !flipped ? d->r * d->s : 0;
    RN50_REQUIRE(flipped || p.flip_taps, RN50_EUNSUPPORTED, "conv2d_bwd_data: the plan's kernel takes a flipped filter");  // see the caller's choice
    set_planes(p, b.g, planes, ge.Mout, ws, st);
    run_igemm(p, b.g, dx, (float *)ws, bf16_of(d), act_of(d), st);
    return launch_status("conv2d_bwd_data");
}

void rn50::launch_filter_flip_batched(const void *jobs, int njobs, int nblocks, const float *theta, float *wt, hipStream_t st)
{
    hipLaunchKernelGGL(filter_flip_batched_kernel, dim3(nblocks), dim3(256), 0, st, (const FlipJob *)jobs, njobs, theta, wt);
}

void rn50::launch_filter_flip(int K, int C, int RS, const float *w, float *wt, hipStream_t st)
{
    hipLaunchKernelGGL(filter_flip_transpose_kernel, dim3(ceil_div(C, kFlipTile), ceil_div(K, kFlipTile), RS), dim3(256), 0, st, K, C, RS, w, wt);
}

extern "C" int conv2d_bwd_data(const rn50_conv_desc *d, const float *dy, const float *w, float *dx, void *ws,
                               size_t ws_bytes, void *stream)
{
    const ConfigScope snapshot;
    if (int rc = conv_check("conv2d_bwd_data", d)) return rc;
    RN50_REQUIRE(dy && w && dx, RN50_EINVAL, "conv2d_bwd_data: null pointer");
    RN50_REQUIRE(d->r == d->s, RN50_EUNSUPPORTED, "conv2d_bwd_data: non-square filters are not supported");
    RN50_REQUIRE(aligned16(dy) && aligned16(w) && aligned16(dx) && aligned16(ws), RN50_EINVAL,
                 "conv2d_bwd_data: pointers must be 16-byte aligned");
    RN50_REQUIRE(act_of(d) != 2, RN50_EUNSUPPORTED, "conv2d_bwd_data: RN50_DTYPE_BF16_ACT_F32IN is for the forward pass and the filter gradient");
    Fp32Math math = kFp32Split;
    BwdDataPlan b = plan_bwd_data(d, math);
    while (math != kNoPlanes && ws_bytes < b.wt_bytes + b.part_bytes) b = plan_bwd_data(d, math = less_room(math));  // less room than the query names
    RN50_REQUIRE(ws && ws_bytes >= b.wt_bytes + b.part_bytes, RN50_EWORKSPACE, "conv2d_bwd_data: workspace too small (%zu < %zu)",
                 ws_bytes, b.wt_bytes + b.part_bytes);
    hipStream_t st = (hipStream_t)stream;
    // workspace = [flipped filter][partial tiles]
    char *rest = (char *)ws + b.wt_bytes;
    // the halves' preparation flips as well, and igemm_small_kernel reads the filter as it is
    if (b.g.kind == kHalf || (math != kNoPlanes && small_bwd(d, b, false).grid))
        return conv_bwd_data_pretransposed(math, d, dy, w, dx, rest, ws_bytes - b.wt_bytes, st, nullptr, false);
    float *wt = (float *)ws;
    launch_filter_flip(d->k, d->c, d->r * d->s, w, wt, st);
    return conv_bwd_data_pretransposed(math, d, dy, wt, dx, rest, ws_bytes - b.wt_bytes, st);
}

extern "C" int conv2d_filter_flip(const rn50_conv_desc *d, const float *w, float *wt, void *stream)
{
    if (int rc = conv_check("conv2d_filter_flip", d)) return rc;
    RN50_REQUIRE(w && wt && w != wt, RN50_EINVAL, "conv2d_filter_flip: null pointer or in-place call");
    RN50_REQUIRE(aligned16(w) && aligned16(wt), RN50_EINVAL, "conv2d_filter_flip: pointers must be 16-byte aligned");
    launch_filter_flip(d->k, d->c, d->r * d->s, w, wt, (hipStream_t)stream);
    return launch_status("conv2d_filter_flip");
}

extern "C" int conv2d_bwd_data_flipped(const rn50_conv_desc *d, const float *dy, const float *wt, float *dx, void *ws,
                                       size_t ws_bytes, void *stream)
{
    const ConfigScope snapshot;
    if (int rc = conv_check("conv2d_bwd_data_flipped", d)) return rc;
    RN50_REQUIRE(dy && wt && dx, RN50_EINVAL, "conv2d_bwd_data_flipped: null pointer");
    RN50_REQUIRE(d->r == d->s, RN50_EUNSUPPORTED, "conv2d_bwd_data_flipped: non-square filters are not supported");
    RN50_REQUIRE(aligned16(dy) && aligned16(wt) && aligned16(dx) && aligned16(ws), RN50_EINVAL,
                 "conv2d_bwd_data_flipped: pointers must be 16-byte aligned");
    RN50_REQUIRE(act_of(d) != 2, RN50_EUNSUPPORTED, "conv2d_bwd_data_flipped: RN50_DTYPE_BF16_ACT_F32IN is for the forward pass and the filter gradient");
    Fp32Math math = kFp32Split;
    size_t need = plan_bwd_data(d, math).part_bytes;
    while (math != kNoPlanes && ws_bytes < need) need = plan_bwd_data(d, math = less_room(math)).part_bytes;
    RN50_REQUIRE(ws_bytes >= need && (need == 0 || ws), RN50_EWORKSPACE, "conv2d_bwd_data_flipped: workspace too small (%zu < %zu)",
                 ws_bytes, need);
    return conv_bwd_data_pretransposed(math, d, dy, wt, dx, ws, ws_bytes, (hipStream_t)stream);
}

static int conv_bwd_weight_impl(const char *who, const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift,
                                const float *dy, float *dw, void *ws, size_t ws_bytes, void *stream, Fp32Math math = kFp32Split);

extern "C" int conv2d_bwd_weight(const rn50_conv_desc *d, const float *x, const float *dy, float *dw, void *ws,
                                 size_t ws_bytes, void *stream)
{
    return conv_bwd_weight_impl("conv2d_bwd_weight", d, x, nullptr, nullptr, dy, dw, ws, ws_bytes, stream);
}

extern "C" int conv2d_bwd_weight_bnrelu_input(const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift,
                                              const float *dy, float *dw, void *ws, size_t ws_bytes, void *stream)
{
    RN50_REQUIRE(in_scale && in_shift && aligned16(in_scale) && aligned16(in_shift), RN50_EINVAL,
                 "conv2d_bwd_weight_bnrelu_input: scale and shift must be non-null and 16-byte aligned");
    RN50_REQUIRE(d && d->c % 4 == 0, RN50_EUNSUPPORTED, "conv2d_bwd_weight_bnrelu_input: the channel count must be a multiple of 4");
    return conv_bwd_weight_impl("conv2d_bwd_weight_bnrelu_input", d, x, in_scale, in_shift, dy, dw, ws, ws_bytes, stream);
}

static int conv_bwd_weight_impl(const char *who, const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift,
                                const float *dy, float *dw, void *ws, size_t ws_bytes, void *stream, Fp32Math math)
{
    const ConfigScope snapshot;
    if (int rc = conv_check(who, d)) return rc;
    RN50_REQUIRE(x && dy && dw, RN50_EINVAL, "%s: null pointer", who);
    RN50_REQUIRE(aligned16(x) && aligned16(dy) && aligned16(dw) && aligned16(ws), RN50_EINVAL, "%s: pointers must be 16-byte aligned", who);
    RN50_REQUIRE(d->k % 4 == 0, RN50_EUNSUPPORTED, "%s: K must be a multiple of 4", who);
    const Geom ge = geom(d);
    const bool vec = d->c % 4 == 0;
    const size_t partial = (size_t)d->k * ge.Kdim * sizeof(float);
    const int sgrid = in_scale ? 0 : stem_wgrad_grid(d, ge);
    if (sgrid && (!act_of(d) || ws_bytes >= sgrid * partial)) {
        // the network's first layer has a kernel of its own (input tile and dy tile in LDS, one partial per workgroup)
        const size_t sneed = sgrid * partial;
        RN50_REQUIRE(ws && ws_bytes >= sneed, RN50_EWORKSPACE, "%s: workspace too small (%zu < %zu)", who, ws_bytes, sneed);
        StemWP sp{};
        sp.x = x; sp.dy = dy; sp.part = (float *)ws;
        sp.N = d->n; sp.IH = d->h; sp.IW = d->w; sp.OH = ge.P; sp.OW = ge.Q;
        sp.tiles_h = ceil_div(ge.P, kStemTH); sp.tiles_w = ceil_div(ge.Q, kStemTW);
        sp.ntiles = d->n * sp.tiles_h * sp.tiles_w;
        launch_stem_wgrad(act_of(d) ? 1 : 2, sgrid, sp, (hipStream_t)stream);
        const long scount4 = (long)d->k * ge.Kdim / 4;
        launch_splitk_reduce(scount4, sgrid, (long)d->k * ge.Kdim, (const float *)ws, dw, (hipStream_t)stream);
        return launch_status(who);
    }
    const bool copy = wgrad_is_copy(d);
    GemmPlan pl = copy ? plan_wgrad_copy(d, d->k, ge.Kdim, ge.Mout) : plan_wgrad(d, d->k, ge.Kdim, ge.Mout, math);
    if (pl.terms && ws_bytes < wgrad_bytes(d, pl, ge)) pl = plan_wgrad(d, d->k, ge.Kdim, ge.Mout, kNoHalf);
    if (ws_bytes < pl.split * partial) pl = plan_wgrad(d, d->k, ge.Kdim, ge.Mout, kNoPlanes);  // less room than the query names: another cut
    const size_t need = wgrad_bytes(d, pl, ge);
    RN50_REQUIRE(ws && ws_bytes >= need, RN50_EWORKSPACE, "%s: workspace too small (%zu < %zu)", who, ws_bytes, need);
    RN50_REQUIRE(((long)d->k * ge.Kdim) % 4 == 0, RN50_EUNSUPPORTED, "%s: filter size must be a multiple of 4", who);
    const int act = act_of(d);
    RN50_REQUIRE(!act || d->k % 8 == 0, RN50_EUNSUPPORTED, "%s: with bf16 activations K must be a multiple of 8", who);
    RN50_REQUIRE(act != 1 || d->c % 8 == 0, RN50_EUNSUPPORTED, "%s: with bf16 activations C must be a multiple of 8", who);
    RN50_REQUIRE(!in_scale || act != 2, RN50_EUNSUPPORTED, "%s: the fused input transform needs an input of the variant's own type", who);
    WgradP p{};
    p.dy = dy; p.x = x; p.out = (float *)ws; p.in_scale = in_scale; p.in_shift = in_shift;
    wgrad_fill(p, d, ge.P, ge.Q, pl.bm, pl.bn, pl.split, pl.chunks_per_split);
    const int grid = p.tiles_k * p.tiles_j * pl.split;
    hipStream_t st = (hipStream_t)stream;
    const bool bf16 = bf16_of(d);
    if (pl.terms) {
        const WgradTermsRoom room = wgrad_terms_room(d, pl, d->k, ge.Kdim, ge.Mout);
        TermsPrep q{};
        q.in_scale = in_scale;
        q.in_shift = in_shift;
        for (int i = 0; i < 2; ++i) {
            q.src[i] = i ? dy : x;
            q.dst[i] = (char *)ws + room.terms[i];
            q.n8[i] = (unsigned)((i ? ge.Mout * d->k : ge.Min * d->c) / 8);
            q.blocks[i] = std::min(2048, ceil_div(q.n8[i], 512));
            q.div8[i] = make_fastdiv((i ? d->k : d->c) / 8);
        }
        p.x_terms = q.dst[0];
        p.dy_terms = q.dst[1];
        launch_terms_prep(q, st);
        launch_wgrad_terms(pl.bm, pl.bn, grid, p, st);
    } else if (pl.products) {
        launch_wgrad_split(pl.bm, pl.bn, grid, p, st);
    } else if (copy) {
        launch_wgrad_act_copy(pl.bm, pl.bn, grid, p, st);
    } else if (act) {  // 64x64 tiles (plan_wgrad keeps to them)
        hipLaunchKernelGGL(wgrad_act_kernel, dim3(grid), dim3(kConvThreads), 0, st, p);
    } else {
#define RN50_WG(BM_, BN_)                                                                                              \
    do {                                                                                                               \
        if (in_scale && bf16) hipLaunchKernelGGL((wgrad_kernel<BM_, BN_, true, true, true>), dim3(grid), dim3(kConvThreads), 0, st, p); \
        else if (in_scale) hipLaunchKernelGGL((wgrad_kernel<BM_, BN_, true, false, true>), dim3(grid), dim3(kConvThreads), 0, st, p);   \
        else if (bf16 && vec) hipLaunchKernelGGL((wgrad_kernel<BM_, BN_, true, true>), dim3(grid), dim3(kConvThreads), 0, st, p);   \
        else if (bf16) hipLaunchKernelGGL((wgrad_kernel<BM_, BN_, false, true>), dim3(grid), dim3(kConvThreads), 0, st, p);    \
        else if (vec) hipLaunchKernelGGL((wgrad_kernel<BM_, BN_, true, false>), dim3(grid), dim3(kConvThreads), 0, st, p);     \
        else hipLaunchKernelGGL((wgrad_kernel<BM_, BN_, false, false>), dim3(grid), dim3(kConvThreads), 0, st, p);             \
    } while (0)
    if (pl.bm == 128 && pl.bn == 128) RN50_WG(128, 128);
    else if (pl.bm == 128) RN50_WG(128, 64);
    else if (pl.bn == 128) RN50_WG(64, 128);
    else RN50_WG(64, 64);
#undef RN50_WG
    }
    const long count4 = p.split_stride / 4;
    launch_splitk_reduce(count4, pl.split, p.split_stride, (const float *)ws, dw, st);
    return launch_status(who);
}

int rn50::conv_bwd_weight_math(Fp32Math math, const rn50_conv_desc *d, const float *x, const float *in_scale, const float *in_shift, const float *dy,
                               float *dw, void *ws, size_t ws_bytes, hipStream_t st)
{
    return conv_bwd_weight_impl("conv2d_bwd_weight", d, x, in_scale, in_shift, dy, dw, ws, ws_bytes, st, math);
}
