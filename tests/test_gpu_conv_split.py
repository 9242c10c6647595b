"""fp32 convolutions on the bf16 matrix instruction: every operand, times 2^16, is the exact sum of three bf16 terms.  What that could break
and a plain comparison at the usual bar would not show: precision below the bar, operands that have no finite split, magnitudes
whose small terms leave the bf16 range.  References: float64 on the CPU from the same fp32 operands."""
import numpy as np
import pytest
import torch

from paper_1711_04325_amd import binding as rn
from tests.gpu_util import empty, ws_bytes

pytestmark = pytest.mark.gpu

# (n, c, h, k, r, stride, pad): vector and scalar gathers, ragged row and column tiles, strided data gradients of both kinds
CASES = [(2, 64, 14, 64, 3, 1, 1), (1, 32, 9, 68, 1, 1, 0), (3, 96, 13, 160, 3, 2, 1), (2, 20, 11, 24, 3, 1, 1), (2, 128, 8, 64, 1, 2, 0),
         (4, 256, 7, 256, 3, 1, 1), (2, 64, 16, 128, 3, 2, 1)]


def _conv64(x, w, stride, pad):
    return torch.nn.functional.conv2d(x.double().permute(0, 3, 1, 2), w.double().permute(0, 3, 1, 2), stride=stride, padding=pad).permute(0, 2, 3, 1)


def _dx64(dy, w, stride, pad, h):
    return torch.nn.grad.conv2d_input((dy.shape[0], w.shape[3], h, h), w.double().permute(0, 3, 1, 2), dy.double().permute(0, 3, 1, 2), stride,
                                      pad).permute(0, 2, 3, 1)


def _dw64(x, dy, r, stride, pad):
    return torch.nn.grad.conv2d_weight(x.double().permute(0, 3, 1, 2), (dy.shape[3], x.shape[3], r, r), dy.double().permute(0, 3, 1, 2), stride,
                                       pad).permute(0, 2, 3, 1)


def _operands(case, seed, scale=1.0):
    n, c, h, k, r, stride, pad = case
    g = torch.Generator().manual_seed(seed)
    p = (h + 2 * pad - r) // stride + 1
    x, dy = torch.randn(n, h, h, c, generator=g) * scale, torch.randn(n, p, p, k, generator=g) * scale
    return x, torch.randn(k, r, r, c, generator=g) * (2.0 / (c * r * r)) ** 0.5, dy


def _device(case, x, w, dy, plan=None):
    """Forward output, data gradient, filter gradient.  Calls this small run on the fp32 instruction by themselves in the first two; with a
    given plan every call runs with split operands."""
    if plan:
        rn.rn50_set_option("igemm_plan", plan)
    try:
        return _run(case, x, w, dy)
    finally:
        rn.rn50_set_option("igemm_plan", None)


def _run(case, x, w, dy):
    n, c, h, k, r, stride, pad = case
    d = rn.conv_desc(n, c, h, h, k, r, r, stride, pad)
    dx_, dw_, ddy = x.cuda(), w.cuda(), dy.cuda()
    y, dx, dw = torch.full_like(ddy, 7.0), torch.full_like(dx_, 7.0), torch.full_like(dw_, 7.0)
    rn.conv2d_fwd(d, dx_, dw_, y, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD)))
    rn.conv2d_bwd_data(d, ddy, dw_, dx, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_DATA)))
    rn.conv2d_bwd_weight(d, dx_, ddy, dw, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_WEIGHT)))
    torch.cuda.synchronize()
    return y.cpu(), dx.cpu(), dw.cpu()


# 1e-30: every term of a split is a normal number; smaller operands: test_precision_at_the_bottom_of_the_range
@pytest.mark.parametrize("plan", [None, "64,64,2", "128,64,1"])
@pytest.mark.parametrize("scale", [1.0, 1e-30, 1e25])
@pytest.mark.parametrize("case", CASES)
def test_precision_is_that_of_fp32_sums(case, scale, plan):
    """One rounding of a sum of up to 16 products at a time: rms error of L/16 roundings of 2^-25 of the growing sum, below
    2^-25 * sqrt(L/16) * 2; the longest reduction here (2304) gives 7e-7.  The bar is 8e-7 for all (fp32 sums product by product
    would need 2e-6)."""
    n, c, h, k, r, stride, pad = case
    x, w, dy = _operands(case, 11 + sum(case), scale)
    got = _device(case, x, w, dy, plan)
    if scale != 1.0:
        got = got[:2]   # the filter gradient multiplies two scaled tensors: out of range by design
    refs = (_conv64(x, w, stride, pad), _dx64(dy, w, stride, pad, h), _dw64(x, dy, r, stride, pad))
    for what, a, b in zip(("fwd", "bwd_data", "bwd_weight"), got, refs):
        err = ((a.double() - b).norm() / b.norm()).item()
        assert err <= 8e-7, "%s %s scale %g: %.2e" % (what, case, scale, err)


@pytest.mark.parametrize("plan", [None, "64,64,2", "128,64,1"])
@pytest.mark.parametrize("small", ["x and dy", "w"])
@pytest.mark.parametrize("scale", [2.0 ** -112, 1e-36, 2.0 ** -125])
@pytest.mark.parametrize("case", CASES)
def test_precision_at_the_bottom_of_the_range(case, scale, small, plan):
    """Operands whose low bits lie below the smallest bf16 number (2^-112: a few of them, 1e-36: all, 2^-125: subnormal operands too).
    The bar is that of the test above; results are rounded to 2^-149, at 2^-126 to an rms of 4e-8 of them."""
    n, c, h, k, r, stride, pad = case
    x, w, dy = _operands(case, 31 + sum(case), scale if small != "w" else 1.0)
    if small == "w":
        w = w * scale
    y, dx, _ = _device(case, x, w, dy, plan)
    dw = _device(case, x, w, dy / scale, plan)[2] if small != "w" else None   # one small factor only
    refs = {"fwd": (y, _conv64(x, w, stride, pad)), "bwd_data": (dx, _dx64(dy, w, stride, pad, h))}
    if dw is not None:
        refs["bwd_weight"] = (dw, _dw64(x, dy / scale, r, stride, pad))
    for what, (a, b) in refs.items():
        err = ((a.double() - b).norm() / b.norm()).item()
        assert err <= 8e-7, "%s %s %s %g: %.2e" % (what, case, small, scale, err)


# (n, c, h, k, r), the errors of the fp32 instruction in the plan it has for that call, behind a BN's backward pass and for operands of
# one sign, each plus 5 % for other draws: calls on both sides of the rule that sends them to split operands
LONG = [((128, 256, 14, 256, 3), 4.6e-7, 8.0e-8), ((16, 128, 64, 144, 1), 4.2e-7, 6.1e-8), ((64, 512, 28, 128, 1), 3.7e-7, 6.6e-8),
        ((64, 128, 28, 128, 3), 4.8e-7, 7.0e-8), ((64, 512, 32, 512, 3), 1.97e-6, 7.0e-7), ((2, 64, 56, 256, 1), 2.1e-7, 6.3e-8)]


@pytest.mark.parametrize("case,bar,bar_one_sign", LONG)
def test_filter_gradients_over_many_pixels_are_as_precise_as_on_the_fp32_instruction(case, bar, bar_one_sign):
    n, c, h, k, r = case
    g = torch.Generator(device="cuda").manual_seed(sum(case))
    x = torch.randn(n, h, h, c, generator=g, device="cuda").relu_()
    # what a BN + ReLU passes back: half of the gradient is zero before the BN, small and of one sign behind it
    y = torch.randn(n * h * h, k, generator=g, device="cuda")
    dz = torch.randn(n * h * h, k, generator=g, device="cuda") * 0.01 * (y > 0)
    dy = (dz - dz.mean(0) - y * (dz * y).mean(0)).reshape(n, h, h, k)
    del dz, y
    ck, cc = min(k, 64), min(c, 64)   # the reference covers 64 x 64 filter channels, in float64 on the GPU
    xp = torch.nn.functional.pad(x[..., :cc].double(), (0, 0, r // 2, r // 2, r // 2, r // 2))
    d = rn.conv_desc(n, c, h, h, k, r, r, 1, r // 2)
    ws = ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_WEIGHT))
    for what, grad, limit in (("BN", dy, bar), ("one sign", dy.abs(), bar_one_sign)):
        dw = torch.full((k, r, r, c), 7.0, device="cuda")
        rn.conv2d_bwd_weight(d, x, grad, dw, ws)
        flat = grad[..., :ck].double().reshape(-1, ck).t().contiguous()
        ref = torch.stack([torch.stack([flat @ xp[:, i:i + h, j:j + h, :].reshape(-1, cc) for j in range(r)], 1) for i in range(r)], 1)
        err = ((dw[:ck, :, :, :cc].double() - ref).norm() / ref.norm()).item()
        assert err <= limit, "%s %s: %.2e" % (what, case, err)


# (n, c, h, k, r, stride, pad): either side of the lines where a call changes its instruction: 256 and 272 workgroups; channels gathered one
# by one with 64-row tiles and with 128-row tiles
@pytest.mark.parametrize("case", [(16, 64, 16, 256, 1, 1, 0), (17, 64, 16, 256, 1, 1, 0), (40, 40, 28, 64, 1, 1, 0), (54, 40, 56, 104, 1, 1, 0)])
def test_both_sides_of_the_choice_of_instruction(case):
    """The bar of the fp32 instruction: 2^-25 * sqrt(L/2) * 2 for sums of up to 256 products."""
    n, c, h, k, r, stride, pad = case
    x, w, dy = _operands(case, 41 + sum(case))
    y, dx, _ = _run(case, x, w, dy)
    for what, a, b in (("fwd", y, _conv64(x, w, stride, pad)), ("bwd_data", dx, _dx64(dy, w, stride, pad, h))):
        assert ((a.double() - b).norm() / b.norm()).item() <= 7e-7, what


@pytest.mark.parametrize("plan", [None, "128,128,1", "64,64,3"])
@pytest.mark.parametrize("case", CASES)
def test_values_without_a_finite_split(case, plan):
    """Infinities, NaNs and numbers that round to infinity in bf16 (3.39e38 .. 3.4028e38) give what fp32 arithmetic gives:
    infinities stay infinities of their sign, NaN only where infinities of both signs or a NaN meet, and every output
    that the value does not touch is what it was."""
    n, c, h, k, r, stride, pad = case
    x, w, dy = _operands(case, 23 + sum(case))
    x[0, 1, 2, 3], x[n - 1, h - 1, h - 1, c - 1], x[0, h - 1, 0, 5], x[0, 3, 3, 1] = np.inf, -np.inf, np.nan, 3.4e38
    dy[0, 0, 0, 2], dy[n - 1, -1, -1, k - 1], dy[0, -1, 0, 7] = np.inf, -np.inf, np.nan
    w[k - 1, 0, 0, 0] = np.inf
    if plan:
        rn.rn50_set_option("igemm_plan", plan)
        rn.rn50_set_option("wgrad_plan", plan)
    try:
        y, dx, dw = _device(case, x, w, dy)
    finally:
        rn.rn50_set_option("igemm_plan", None)
        rn.rn50_set_option("wgrad_plan", None)
    # float64 sums of the same operands; beyond the fp32 range they are infinities in fp32.  Padding multiplies as a zero on both
    # sides, so an infinite weight makes NaNs along the border.
    for what, got, ref in (("fwd", y, _conv64(x, w, stride, pad)), ("bwd_weight", dw, _dw64(x, dy, r, stride, pad))):
        ref32 = ref.float()
        fine = torch.isfinite(ref32) & (ref.abs() < 1e38)
        assert torch.equal(torch.isfinite(got)[fine], fine[fine]), what
        ok = fine & (ref.abs() < 1e30)
        err = ((got.double() - ref)[ok].norm() / ref[ok].norm()).item()
        assert err <= 8e-7, "%s: %.2e" % (what, err)
        both = torch.isinf(ref32) & torch.isinf(ref)
        assert torch.equal(got[both], ref32[both]), what      # signed infinities
        assert torch.isnan(got[torch.isnan(ref32)]).all(), what
    # the data gradient: elements that no special value reaches (the infinite weight touches input channel 0 of the border too)
    ref = _dx64(dy, w, stride, pad, h)
    assert torch.isnan(dx[torch.isnan(ref)]).all()
    fine = torch.isfinite(ref)
    fine[..., 0] = False
    assert torch.isfinite(dx[fine]).all() and ((dx.double() - ref)[fine].norm() / ref[fine].norm()).item() <= 8e-7
    both = torch.isinf(ref)
    both[..., 0] = False
    assert torch.equal(dx.double()[both], ref[both])
