"""fp32 convolutions both of whose operands are prepared beforehand: forward pass and data gradient as fp16 halves, filter gradient split
into bf16 terms.  Rows of "operand_plans" send small calls there: tiles that end in the middle of rows, columns and reduction, strides,
padding, the scattered data gradient, pieces of the reduction.  References: float64 on the CPU from the same fp32 operands."""
import pytest
import torch

from paper_1711_04325_amd import binding as rn
from tests.gpu_util import ws_bytes

pytestmark = pytest.mark.gpu
# (n, c, h, k, r, stride): one stage to a tap and several, fewer rows and columns than a tile, 33 x 33 pixels, the largest filter (25 taps)
CASES = [(2, 32, 7, 32, 1, 1), (1, 64, 9, 68, 3, 1), (3, 96, 13, 160, 3, 2), (2, 64, 15, 128, 1, 2), (2, 128, 8, 64, 1, 2), (1, 32, 33, 96, 5, 1), (5, 160, 6, 224, 3, 1)]
PLANS = ["64,64,1", "64,128,3", "128,64,2"]
# half_bar: what the halves drop is 9e-8 of normal operands (1.1e-7 with the sums), at most 2^-23 + 2^-22 of each product where all of it
# adds up; bf16 terms: see test_gpu_conv_split
HALF_BAR, TERMS_BAR = 4e-7, 8e-7


def _operands(case, seed):
    n, c, h, k, r, stride = case
    g = torch.Generator().manual_seed(seed)
    p = (h + 2 * (r // 2) - r) // stride + 1
    return torch.randn(n, h, h, c, generator=g), torch.randn(k, r, r, c, generator=g) * (2.0 / (c * r * r)) ** 0.5, torch.randn(n, p, p, k, generator=g)


def _refs(case, x, w, dy):
    n, c, h, k, r, stride = case
    x, w, dy = (t.double().permute(0, 3, 1, 2) for t in (x, w, dy))
    return {"fwd": torch.nn.functional.conv2d(x, w, stride=stride, padding=r // 2).permute(0, 2, 3, 1),
            "bwd_data": torch.nn.grad.conv2d_input((n, c, h, h), w, dy, stride, r // 2).permute(0, 2, 3, 1),
            "bwd_weight": torch.nn.grad.conv2d_weight(x, (k, c, r, r), dy, stride, r // 2).permute(0, 2, 3, 1)}


def _run(case, plan, x, w, dy, fused=None, only=("fwd", "bwd_data", "bwd_weight")):
    n, c, h, k, r, stride = case
    d = rn.conv_desc(n, c, h, h, k, r, r, stride, r // 2)
    ops = {"fwd": rn.OP_FWD, "bwd_data": rn.OP_BWD_DATA, "bwd_weight": rn.OP_BWD_WEIGHT}
    if k % 32:   # a gathered dy needs whole groups of 32 channels
        only = [o for o in only if o == "fwd"]
    if stride == 2 and (r > 1 or h % 2):   # a dilated gather keeps its kernel
        only = [o for o in only if o != "bwd_data"]
    rn.rn50_set_option("operand_plans", ";".join("%d,%d,%d,%d,%d,%d,%d,%d,%s" % (ops[o], n, c, h, k, r, stride, r // 2, plan) for o in only))
    x, w, dy = x.cuda(), w.cuda(), dy.cuda()
    out = {"fwd": torch.full_like(dy, 7.0), "bwd_data": torch.full_like(x, 7.0), "bwd_weight": torch.full_like(w, 7.0)}
    try:
        for o in only:
            need = rn.rn50_conv_workspace_bytes(d, ops[o])
            bm, bn, _, _ = rn.rn50_conv_plan(d, ops[o])
            assert "%d,%d" % (bm, bn) == plan.rsplit(",", 1)[0]
            room = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
            ws = room[:need]
            if o == "fwd":
                rn.conv2d_fwd(d, x, w, out[o], ws) if fused is None else rn.conv2d_fwd_bnrelu_input(d, x, *fused, w, out[o], ws)
            elif o == "bwd_data":
                rn.conv2d_bwd_data(d, dy, w, out[o], ws)
                wt, flipped = torch.empty(r * r * c * k, device="cuda"), torch.full_like(x, 7.0)
                rn.conv2d_filter_flip(d, w, wt)
                rn.conv2d_bwd_data_flipped(d, dy, wt, flipped, ws_bytes(need))
                assert torch.equal(flipped.view(torch.int32), out[o].view(torch.int32))   # the preparation flips as the flip does
            else:
                rn.conv2d_bwd_weight(d, x, dy, out[o], ws) if fused is None else rn.conv2d_bwd_weight_bnrelu_input(d, x, *fused, dy, out[o], ws)
            torch.cuda.synchronize()
            assert (room[need:] == 0x5A).all()
    finally:
        rn.rn50_set_option("operand_plans", None)
    return {o: out[o].cpu() for o in only}


def _bar(o):
    return TERMS_BAR if o == "bwd_weight" else HALF_BAR


def _err(a, b):
    return ((a.double() - b).norm() / b.norm()).item()


@pytest.mark.parametrize("plan", PLANS)
@pytest.mark.parametrize("case", CASES)
def test_every_tile(case, plan):
    x, w, dy = _operands(case, 3 + sum(case))
    refs = _refs(case, x, w, dy)
    for o, got in _run(case, plan, x, w, dy).items():
        assert _err(got, refs[o]) <= _bar(o), (o, _err(got, refs[o]))


@pytest.mark.parametrize("case", [CASES[2], CASES[6]])
def test_fused_input(case):
    n, c = case[:2]
    x, w, dy = _operands(case, 5 + sum(case))
    g = torch.Generator().manual_seed(c)
    scale, shift = torch.rand(c, generator=g) + 0.5, torch.randn(c, generator=g) * 0.3
    z = (x.double() * scale.double() + shift.double()).float().relu()   # one rounding, as of the fused multiply-add
    refs = _refs(case, z, w, dy)
    for o, got in _run(case, PLANS[1], x, w, dy, (scale.cuda(), shift.cuda()), ("fwd", "bwd_weight")).items():
        assert _err(got, refs[o]) <= _bar(o), (o, _err(got, refs[o]))


@pytest.mark.parametrize("plan", PLANS)
def test_batch_statistics(plan):
    n, c, h, k, r, stride = case = (3, 64, 11, 100, 3, 1)   # 363 rows: whole tiles and one that ends inside
    x, w, _ = _operands(case, 8)
    d = rn.conv_desc(n, c, h, h, k, r, r, stride, 1)
    gamma, beta = torch.ones(k).cuda(), torch.zeros(k).cuda()
    rn.rn50_set_option("operand_plans", "%d,%d,%d,%d,%d,%d,%d,%d,%s" % (rn.OP_FWD, n, c, h, k, r, stride, 1, plan))
    try:
        y, vec = torch.empty(n, h, h, k).cuda(), [torch.empty(k).cuda() for _ in range(4)]
        rn.conv2d_fwd_bnstats(d, x.cuda(), None, None, w.cuda(), y, gamma, beta, 2e-5, *vec, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD_BNSTATS)))
        torch.cuda.synchronize()
    finally:
        rn.rn50_set_option("operand_plans", None)
    f = y.double().cpu().reshape(-1, k)
    mean, invstd = f.mean(0), 1 / torch.sqrt(f.var(0, unbiased=False) + 2e-5)
    assert (vec[0].double().cpu() - mean).abs().max() <= 1e-6 * f.std() and ((vec[1].double().cpu() - invstd) / invstd).abs().max() <= 1e-6


@pytest.mark.parametrize("sx,sw", [(2.0 ** -140, 1.0), (1.0, 2.0 ** -140), (2.0 ** 100, 2.0 ** -20), (2.0 ** -60, 2.0 ** 110), (2.0 ** -70, 2.0 ** -70)])
def test_magnitudes(sx, sw):
    """Tensors at the bottom (numbers below 2^-126 have fewer bits themselves: the reference is of the numbers as they are) and the top of
    the range, and results that are subnormal: a power of two moves a tensor where fp16 holds it, and the sums back."""
    case = CASES[6]
    x, w, dy = _operands(case, 21)
    x, dy, w = x * sx, dy * sx, w * sw
    refs = _refs(case, x, w, dy)
    for o, got in _run(case, PLANS[0], x, w, dy, only=("fwd", "bwd_data")).items():
        want = refs[o]
        off = ((got.double() - want).norm() / want.norm()).item()
        # results are rounded to multiples of 2^-149
        assert off <= HALF_BAR + 2.0 ** -150 * want.numel() ** 0.5 / want.norm().item(), (o, off)


@pytest.mark.parametrize("what", ["image", "rows", "filter", "pixel"])
def test_small_beside_large(what):
    """What is small beside the rest of its tensor keeps its precision where nothing else reaches it: below 2^-27 of the largest number the
    halves do not hold 24 bits, and the outputs are formed again on the fp32 instruction, which rounds the sum of 1440 products at every other: an
    rms error of 2^-24/sqrt(3) * sqrt(720/2) = 6.5e-7 of normal operands, a fifth more for other draws."""
    case = n, c, h, k, r, stride = CASES[6]
    x, w, dy = _operands(case, 23)
    s = 2.0 ** -60
    if what == "image":
        x[3] *= s
        part = (3,)
    elif what == "rows":    # output row 5 sees input rows 4 and 5
        x[2, 4:] *= s
        part = (2, 5)
    elif what == "filter":
        w[17] *= s
        part = (slice(None), slice(None), slice(None), 17)
    else:
        x[1, 2:5, 1:4] *= s
        part = (1, 3, 2)
    refs = _refs(case, x, w, dy)
    for plan in PLANS:
        got = _run(case, plan, x, w, dy, only=("fwd",))["fwd"]
        assert _err(got, refs["fwd"]) <= 8e-7 and _err(got[part], refs["fwd"][part]) <= 8e-7, (plan, _err(got[part], refs["fwd"][part]))


# A channel of large numbers hides nothing of the others where its weights are zero or as small: 2^-27 of the largest number and below, the halves
# hold fewer than 24 bits, below 2^-52 none.  Formed again, a sum of 1440 products on the fp32 instruction in parts of 128: the parts' sums round at every
# other product, 2^-24/sqrt(3) * sqrt(64), a dozen additions of the parts 2^-24/sqrt(3) * sqrt(12/2) more: 2.9e-7, a third more for other draws.
AGAIN_BAR = 3.9e-7


@pytest.mark.parametrize("b", [28, 32, 40, 56, 100])
@pytest.mark.parametrize("what", ["zero", "inverse", "one row", "filter"])
def test_channels_of_other_scales(what, b):
    case = n, c, h, k, r, stride = CASES[6]
    x, w, dy = _operands(case, 29)
    g = torch.Generator().manual_seed(b)
    if what == "zero":          # one channel of each group of 32, without weights
        x[..., 3::32] *= 2.0 ** b
        w[..., 3::32] = 0
        dy[..., 5::32] *= 2.0 ** b
        w[5::32] = 0
    elif what == "inverse":     # every channel a scale of its own, its weights the inverse: all products count alike
        e, f = torch.randint(0, b + 1, (c,), generator=g).float(), torch.randint(0, b + 1, (k,), generator=g).float()
        x, dy, w = x * 2.0 ** e, dy * 2.0 ** f, w * 2.0 ** -e * 2.0 ** -f.reshape(k, 1, 1, 1)
    elif what == "one row":     # large beside them in the same block: the outputs of every other filter row and channel
        x[..., 3] *= 2.0 ** b
        w[17, :, :, 3] = 0
        dy[..., 5] *= 2.0 ** b
        w[5, :, :, 19] = 0
    else:                       # the filter's numbers are the large ones
        w[1:, :, :, 3] *= 2.0 ** b
        x[..., 3] = 0
        w[5, :, :, 4:] *= 2.0 ** b
        dy[..., 5] = 0
    refs = _refs(case, x, w, dy)
    for plan in PLANS:
        for o, got in _run(case, plan, x, w, dy, only=("fwd", "bwd_data")).items():
            ref = refs[o]
            if what == "inverse":   # outputs have their channels' scales: each channel by itself
                for ch in range(got.shape[-1]):
                    assert _err(got[..., ch], ref[..., ch]) <= 2 * AGAIN_BAR, (plan, o, ch, _err(got[..., ch], ref[..., ch]))   # 180 and fewer outputs
                continue
            if what == "one row":
                ch = 17 if o == "fwd" else 19
                assert _err(got[..., ch], ref[..., ch]) <= 2 * AGAIN_BAR, (plan, o, _err(got[..., ch], ref[..., ch]))
            elif what == "filter" and o == "bwd_data":   # channel 3's weights are the large ones
                assert _err(got[..., 3], ref[..., 3]) <= 2 * AGAIN_BAR
                keep = [i for i in range(c) if i != 3]
                got, ref = got[..., keep], ref[..., keep]
            assert _err(got, ref) <= AGAIN_BAR, (plan, o, _err(got, ref))


def test_zeros_and_a_single_number():
    case = n, c, h, k, r, stride = CASES[6]
    x, w, dy = _operands(case, 25)
    got = _run(case, PLANS[0], x * 0, w, dy * 0)
    assert all((t == 0).all() for t in got.values())
    x = x * 0
    x[4, 5, 5, 31] = 3e-39
    got = _run(case, PLANS[2], x, w, dy, only=("fwd",))["fwd"].double()
    assert (got - _refs(case, x, w, dy)["fwd"]).abs().max() <= 2.0 ** -149


@pytest.mark.parametrize("plan", PLANS)
def test_values_without_halves(plan):
    """Infinities, a NaN and a number next to the largest reach the outputs that fp32 arithmetic would let them reach, and no others."""
    case = n, c, h, k, r, stride = CASES[6]
    x, w, dy = _operands(case, 27)
    x[0, 1, 2, 3], x[1, 5, 5, 159], x[2, 3, 0, 5], x[3, 5, 4, 7] = float("inf"), float("-inf"), float("nan"), 3.4e38
    dy[4, 2, 2, 100] = float("inf")
    refs = _refs(case, x, w, dy)
    for o, got in _run(case, plan, x, w, dy).items():
        ref = refs[o]
        assert torch.isnan(got[torch.isnan(ref)]).all() and torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)].float()), o
        fine = torch.isfinite(ref) & (ref.abs() < 1e30)
        assert fine.any() and torch.isfinite(got[fine]).all() and ((got.double() - ref)[fine].norm() / ref[fine].norm()).item() <= 1.5e-6, o


@pytest.mark.parametrize("op", ["fwd", "bwd_data"])
def test_option_for_operands_of_mostly_zeros(op):
    """Halves drop bits whatever the operands, six bf16 products next to none: half_products = 0 keeps a call on the latter.  Bars: the largest of 14 calls
    measured, a tenth more for other draws; a number that is copied loses up to 2^-23 in halves."""
    n, c, h, k, r = 16, 128, 28, 128, 3
    o = rn.OP_FWD if op == "fwd" else rn.OP_BWD_DATA
    g = torch.Generator().manual_seed(61)
    x = torch.randn(n, h, h, c, generator=g) * (torch.rand(n, h, h, c, generator=g) < 0.1)
    w, same = torch.randn(k, r, r, c, generator=g) * (2.0 / (c * r * r)) ** 0.5, torch.zeros(k, r, r, c)
    same[:, 1, 1] = torch.eye(c)
    d = rn.conv_desc(n, c, h, h, k, r, r, 1, 1)
    ref = _refs((n, c, h, k, r, 1), x, w, x)[op]
    ws = ws_bytes(64 << 20)
    err, copy = {}, {}
    for option in ("0", "3"):
        rn.rn50_set_option("half_products", option)
        try:
            assert rn.rn50_conv_workspace_bytes(d, o) <= ws.numel()
            for f in (w, same):
                out = torch.full_like(x, 7.0).cuda()
                (rn.conv2d_fwd if op == "fwd" else rn.conv2d_bwd_data)(d, x.cuda(), f.cuda(), out, ws)
                (err if f is w else copy)[option] = out.cpu()
        finally:
            rn.rn50_set_option("half_products", None)
    assert torch.equal(copy["0"], x) and not torch.equal(copy["3"], x) and ((copy["3"] - x).abs() <= 2.0 ** -23 * x.abs()).all()
    assert _err(err["0"], ref) <= 9.0e-8 and _err(err["3"], ref) <= 1.24e-7


# ---- calls that do not fill the chip (igemm_small_kernel) ----------------------------------------------------------------------------------
SMALL = ["16,16,1", "32,16,1", "16,32,1", "32,32,1"]
# sums of a 16th of the reduction or less on the fp32 instruction (1440 / 16 products, rounded at every other: 2e-7), then five additions
SMALL_BAR = 5e-7


@pytest.mark.parametrize("plan", SMALL)
@pytest.mark.parametrize("case", CASES)
def test_small_calls(case, plan):
    """Ragged rows and columns, fewer stages than wavefronts, strides, the scattered data gradient, flipped filters read as they are."""
    n, c, h, k, r, stride = case
    x, w, dy = _operands(case, 40 + sum(case))
    g = torch.Generator().manual_seed(c)
    scale, shift = torch.rand(c, generator=g) + 0.5, torch.randn(c, generator=g) * 0.3
    z = (x.double() * scale.double() + shift.double()).float().relu()
    refs, fused_ref = _refs(case, x, w, dy), _refs(case, z, w, dy)["fwd"]
    d = rn.conv_desc(n, c, h, h, k, r, r, stride, r // 2)
    rn.rn50_set_option("small_plans", ";".join("%d,%d,%d,%d,%d,%d,%d,%d,%s" % (o, n, c, h, k, r, stride, r // 2, plan) for o in (rn.OP_FWD, rn.OP_BWD_DATA)))
    try:
        assert "%d,%d" % rn.rn50_conv_plan(d, rn.OP_FWD)[:2] == plan[:-2]   # the kernel named here runs
        small = k % 32 == 0 and (stride == 1 or (r == 1 and h % 2 == 0))
        for op in (rn.OP_BWD_DATA, rn.OP_BWD_DATA_FLIPPED):
            assert ("%d,%d" % rn.rn50_conv_plan(d, op)[:2] == plan[:-2]) == small
        fx, fw, fdy = x.cuda(), w.cuda(), dy.cuda()
        y, yf, dx, dxf, ys = (torch.full_like(t, 7.0) for t in (fdy, fdy, fx, fx, fdy))
        ws = ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD_BNSTATS) + rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_DATA))
        rn.conv2d_fwd(d, fx, fw, y, ws)
        rn.conv2d_fwd_bnrelu_input(d, fx, scale.cuda(), shift.cuda(), fw, yf, ws)
        rn.conv2d_bwd_data(d, fdy, fw, dx, ws)
        wt = torch.empty(r * r * c * k, device="cuda")
        rn.conv2d_filter_flip(d, fw, wt)
        rn.conv2d_bwd_data_flipped(d, fdy, wt, dxf, ws)
        vec, ones, zeros = [torch.empty(k).cuda() for _ in range(4)], torch.ones(k).cuda(), torch.zeros(k).cuda()
        rn.conv2d_fwd_bnstats(d, fx, None, None, fw, ys, ones, zeros, 2e-5, *vec, ws)
        torch.cuda.synchronize()
    finally:
        rn.rn50_set_option("small_plans", None)
    assert _err(y.cpu(), refs["fwd"]) <= SMALL_BAR and _err(yf.cpu(), fused_ref) <= SMALL_BAR
    assert torch.equal(ys, y)
    f = y.double().cpu().reshape(-1, k)
    mean, invstd = f.mean(0), 1 / torch.sqrt(f.var(0, unbiased=False) + 2e-5)
    assert (vec[0].double().cpu() - mean).abs().max() <= 1e-6 * f.std() and ((vec[1].double().cpu() - invstd) / invstd).abs().max() <= 1e-6
    if not (stride == 2 and (r > 1 or h % 2)) or k % 32 == 0:
        assert _err(dx.cpu(), refs["bwd_data"]) <= TERMS_BAR and _err(dxf.cpu(), refs["bwd_data"]) <= TERMS_BAR


def test_small_calls_and_infinities():
    case = n, c, h, k, r, stride = CASES[6]
    x, w, dy = _operands(case, 47)
    x[0, 1, 2, 3], x[2, 3, 0, 5], dy[4, 2, 2, 100] = float("inf"), float("nan"), float("-inf")
    refs = _refs(case, x, w, dy)
    d = rn.conv_desc(n, c, h, h, k, r, r, stride, 1)
    for plan in SMALL:
        rn.rn50_set_option("small_plans", ";".join("%d,%d,%d,%d,%d,%d,%d,%d,%s" % (o, n, c, h, k, r, stride, 1, plan) for o in (rn.OP_FWD, rn.OP_BWD_DATA)))
        try:
            y, dx = torch.full_like(dy, 7.0).cuda(), torch.full_like(x, 7.0).cuda()
            rn.conv2d_fwd(d, x.cuda(), w.cuda(), y, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD)))
            rn.conv2d_bwd_data(d, dy.cuda(), w.cuda(), dx, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_DATA)))
        finally:
            rn.rn50_set_option("small_plans", None)
        for got, ref in ((y.cpu(), refs["fwd"]), (dx.cpu(), refs["bwd_data"])):
            assert torch.isnan(got[torch.isnan(ref)]).all() and torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)].float())
            fine = torch.isfinite(ref)
            assert _err(got[fine], ref[fine]) <= SMALL_BAR


# calls that go there by themselves, and what the kernels they went to before left of them (relative error of six bf16 products,
# measured, plus 5 % for other draws)
@pytest.mark.parametrize("case,bars", [((16, 128, 28, 128, 3, 1), (1.61e-7, 2.25e-7, 2.8e-7)), ((32, 256, 14, 512, 3, 1), (1.62e-7, 2.29e-7, 2.41e-7))])
def test_no_less_precise_than_six_products(case, bars):
    n, c, h, k, r, stride = case
    g = torch.Generator(device="cuda").manual_seed(sum(case))
    x = torch.randn(n, h, h, c, generator=g, device="cuda").relu_()
    w = torch.randn(k, r, r, c, generator=g, device="cuda") * (2.0 / (c * r * r)) ** 0.5
    y, dz = torch.randn(n * h * h, k, generator=g, device="cuda"), torch.randn(n * h * h, k, generator=g, device="cuda")
    dz = dz * (y > 0)
    dy = (dz - dz.mean(0) - y * (dz * y).mean(0)).reshape(n, h, h, k)   # behind the backward pass of a BN + ReLU
    d = rn.conv_desc(n, c, h, h, k, r, r, stride, 1)
    out = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    rn.conv2d_fwd(d, x, w, out[0], ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD)))
    rn.conv2d_bwd_data(d, dy, w, out[1], ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_DATA)))
    rn.conv2d_bwd_weight(d, x, dy, out[2], ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_WEIGHT)))
    xp, wd, dyd = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1)), w.double(), dy.double()
    y64, dx64, dw64 = torch.zeros_like(dyd), torch.zeros_like(xp), torch.empty_like(wd)
    for i in range(3):
        for j in range(3):
            t, ws = xp[:, i:i + h, j:j + h], wd[:, i, j].contiguous()
            y64 += (t.reshape(-1, c) @ ws.t().contiguous()).reshape(dyd.shape)
            dx64[:, i:i + h, j:j + h] += (dyd.reshape(-1, k) @ ws).reshape(n, h, h, c)
            dw64[:, i, j] = dyd.reshape(-1, k).t().contiguous() @ t.reshape(-1, c)
    for got, ref, bar in zip(out, (y64, dx64[:, 1:-1, 1:-1], dw64), bars):
        err = ((got.double() - ref).norm() / ref.norm()).item()
        assert err <= bar, (err, bar)
