"""Convolutions whose operands are copied to LDS without registers: filters prepared beforehand (fp32 split into bf16 terms, or
rounded to bf16) and filter gradients of bf16 activations.  Sizes are the smallest that the dispatch sends there, with ragged row,
column and channel tiles; references are float64 on the CPU from the operands as the device has them."""
import pytest
import torch

from paper_1711_04325_amd import binding as rn
from tests.gpu_util import ws_bytes

pytestmark = pytest.mark.gpu
ACT = rn.DTYPE_BF16_ACT

# 5 GFLOP and more: below, a call keeps the kernel that takes the filter as it is
FWD_BWD = [(2, 256, 29, 704, 3, 1, 1),    # odd sizes, 1682 rows, 704 = 5.5 x 128 columns
           (6, 256, 30, 832, 3, 2, 1),    # data gradient by parity classes, skipped taps
           (6, 256, 29, 896, 3, 2, 1),    # ... of an odd input: rows in plain order
           (8, 1088, 31, 640, 1, 1, 0),
           (8, 640, 62, 1088, 1, 2, 0)]   # data gradient scattered over the even positions
PLANS = [None, "128,128,1", "128,64,2", "64,128,1", "64,64,3"]


def _operands(case, seed, dtype):
    n, c, h, k, r, stride, pad = case
    g = torch.Generator().manual_seed(seed)
    p = (h + 2 * pad - r) // stride + 1
    x, dy = torch.randn(n, h, h, c, generator=g).to(dtype), torch.randn(n, p, p, k, generator=g).to(dtype)
    return x, torch.randn(k, r, r, c, generator=g) * (2.0 / (c * r * r)) ** 0.5, dy


def _nchw64(t):
    return t.double().permute(0, 3, 1, 2)


_REF = {}


def _reference(case, act):
    """Operands, and output and data gradient in float64 (once per case; bf16 activations: of the weights as rounded)."""
    if (case, act) not in _REF:
        n, c, h, k, r, stride, pad = case
        x, w, dy = _operands(case, 5 + sum(case), torch.bfloat16 if act else torch.float32)
        wq = w.to(torch.bfloat16).float() if act else w
        y = torch.nn.functional.conv2d(_nchw64(x), _nchw64(wq), stride=stride, padding=pad).permute(0, 2, 3, 1)
        dx = torch.nn.grad.conv2d_input((n, c, h, h), _nchw64(wq), _nchw64(dy), stride, pad).permute(0, 2, 3, 1)
        _REF.clear()
        _REF[case, act] = (x, w, dy, y, dx)
    return _REF[case, act]


def _desc(case, act):
    n, c, h, k, r, stride, pad = case
    return rn.conv_desc(n, c, h, h, k, r, r, stride, pad, in_dtype=ACT) if act else rn.conv_desc(n, c, h, h, k, r, r, stride, pad)


def _err(got, ref):
    return ((got.double().cpu() - ref).norm() / ref.norm()).item()


# fp32: see the bar in test_gpu_conv_split (reductions up to 8064 elements, sqrt(8064 / 2304) times its 8e-7).  bf16 outputs are the
# nearest of 8 bits: off by at most 2^-9 each, so by no more in the norm.
BAR = {False: 1.5e-6, True: 2.0 ** -9 + 1e-5}


@pytest.mark.parametrize("act", [False, True])
@pytest.mark.parametrize("case", FWD_BWD)
def test_prepared_filter(case, act):
    x, w, dy, y_ref, dx_ref = _reference(case, act)
    n, c, h, k, r, stride, pad = case
    d = _desc(case, act)
    fx, fw, fdy = x.cuda(), w.cuda(), dy.cuda()
    for plan in PLANS:
        if plan:
            rows = ["%d,%d,%d,%d,%d,%d,%d,%d,%s" % ((op, n, c, h, k, r, stride, pad, plan)) for op in (rn.OP_FWD, rn.OP_BWD_DATA)]
            rn.rn50_set_option("pre_plans", ";".join(rows))
        try:
            y, dx = torch.full_like(fdy, 7.0), torch.full_like(fx, 7.0)
            rn.conv2d_fwd(d, fx, fw, y, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD)))
            rn.conv2d_bwd_data(d, fdy, fw, dx, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_DATA)))
            torch.cuda.synchronize()
        finally:
            rn.rn50_set_option("pre_plans", None)
        assert _err(y, y_ref) <= BAR[act], (plan, "fwd", _err(y, y_ref))
        assert _err(dx, dx_ref) <= BAR[act], (plan, "bwd_data", _err(dx, dx_ref))


def test_prepared_filter_at_the_bottom_of_the_range():
    """Operands of 1e-36, whose low bits lie below the smallest bf16 number: the input, then the filter."""
    case = FWD_BWD[0]
    x, w, dy, y_ref, dx_ref = _reference(case, False)
    d = _desc(case, False)
    s = 2.0 ** -120   # a power of two: the references scale exactly
    for sx, sw in ((s, 1.0), (1.0, s)):
        y, dx = torch.full_like(dy, 7.0).cuda(), torch.full_like(x, 7.0).cuda()
        rn.conv2d_fwd(d, (x * sx).cuda(), (w * sw).cuda(), y, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD)))
        rn.conv2d_bwd_data(d, (dy * sx).cuda(), (w * sw).cuda(), dx, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_DATA)))
        torch.cuda.synchronize()
        assert _err(y, y_ref * s) <= BAR[False] and _err(dx, dx_ref * s) <= BAR[False], (sx, sw, _err(y, y_ref * s), _err(dx, dx_ref * s))


def test_prepared_filter_and_values_without_a_finite_split():
    """An infinity, a NaN and a number that rounds to infinity in bf16 reach the outputs that fp32 arithmetic would let them reach."""
    case = FWD_BWD[0]
    x, w, dy, y_ref, _ = _reference(case, False)
    x = x.clone()
    x[0, 1, 2, 3], x[1, 28, 28, 255], x[0, 14, 0, 5], x[1, 5, 20, 7] = float("inf"), float("-inf"), float("nan"), 3.4e38
    d = _desc(case, False)
    y = torch.full_like(dy, 7.0).cuda()
    rn.conv2d_fwd(d, x.cuda(), w.cuda(), y, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD)))
    y = y.cpu()
    ref = torch.nn.functional.conv2d(_nchw64(x), _nchw64(w), padding=1).permute(0, 2, 3, 1)
    assert torch.isnan(y[torch.isnan(ref)]).all() and torch.equal(y[torch.isinf(ref)], ref[torch.isinf(ref)].float())
    fine = torch.isfinite(ref) & (ref.abs() < 1e30)
    assert torch.isfinite(y[fine]).all() and ((y.double() - ref)[fine].norm() / ref[fine].norm()).item() <= BAR[False]


@pytest.mark.parametrize("plan", PLANS)
@pytest.mark.parametrize("act", [False, True])
def test_infinite_weight_of_a_tap_that_a_piece_skips(act, plan):
    """Data gradient of a strided 3x3 by parity classes, a whole number of tiles each: an infinite weight at one corner of the filter
    reaches one class only.  In pieces of the reduction none of whose taps reach a class nothing is multiplied, not even zeros."""
    case = n, c, h, k, r, stride, pad = 8, 256, 32, 512, 3, 2, 1
    x, w, dy = _operands(case, 77, torch.bfloat16 if act else torch.float32)
    w[5, 2, 2, 3] = float("inf")
    d = _desc(case, act)
    if plan:
        rn.rn50_set_option("pre_plans", "%d,%d,%d,%d,%d,%d,%d,%d,%s" % (rn.OP_BWD_DATA, n, c, h, k, r, stride, pad, plan))
    try:
        dx = torch.full_like(x, 7.0).cuda()
        rn.conv2d_bwd_data(d, dy.cuda(), w.cuda(), dx, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_DATA)))
        torch.cuda.synchronize()
    finally:
        rn.rn50_set_option("pre_plans", None)
    wq = w.to(torch.bfloat16).double() if act else w.double()
    wq[5, 2, 2, 3] = 0.0
    ref = torch.nn.grad.conv2d_input((n, c, h, h), wq.permute(0, 3, 1, 2), _nchw64(dy), stride, pad).permute(0, 2, 3, 1)
    dx = dx.cpu().double()
    for ph in (0, 1):
        for pw in (0, 1):   # tap (2, 2) reaches the odd rows and columns; the infinity makes channel 3 there infinite
            got, want = dx[:, ph::2, pw::2], ref[:, ph::2, pw::2]
            if (ph, pw) == (1, 1):
                assert not torch.isfinite(got[..., 3]).any()
                got, want = got[..., 4:], want[..., 4:]
            assert torch.isfinite(got).all(), (ph, pw)
            assert ((got - want).norm() / want.norm()).item() <= BAR[act], (ph, pw)


@pytest.mark.parametrize("act", [False, True])
@pytest.mark.parametrize("case", FWD_BWD[:2] + [(2, 64, 14, 64, 3, 1, 1), (128, 256, 14, 1024, 1, 1, 0)])
def test_workspace_limits(case, act):
    """The size a query returns is enough for every call of that operation, flipped filters included; less gives the same values
    from a kernel that needs less, or is refused; nothing is written outside."""
    n, c, h, k, r, stride, pad = case
    d = _desc(case, act)
    x, w, dy = _operands(case, 3, torch.bfloat16 if act else torch.float32)
    fx, fw, fdy = x.cuda(), w.cuda(), dy.cuda()
    wt = torch.empty(r * r * c * k, device="cuda")
    rn.conv2d_filter_flip(d, fw, wt)
    calls = {"fwd": (rn.OP_FWD, fdy, lambda out, ws: rn.conv2d_fwd(d, fx, fw, out, ws)),
             "bwd_data": (rn.OP_BWD_DATA, fx, lambda out, ws: rn.conv2d_bwd_data(d, fdy, fw, out, ws)),
             "flipped": (rn.OP_BWD_DATA_FLIPPED, fx, lambda out, ws: rn.conv2d_bwd_data_flipped(d, fdy, wt, out, ws)),
             "bwd_weight": (rn.OP_BWD_WEIGHT, fw, lambda out, ws: rn.conv2d_bwd_weight(d, fx, fdy, out, ws))}
    for what, (op, like, call) in calls.items():
        need = rn.rn50_conv_workspace_bytes(d, op)
        seen = None
        for size in (need, need - 256, need // 2, 0):
            if size < 0:
                continue
            room = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
            out = torch.full_like(like, 7.0)
            try:
                call(out, room[:size] if size else None)
            except rn.Rn50Error as e:
                assert e.code == rn.EWORKSPACE and size < need, (what, size, need, str(e))
                continue
            torch.cuda.synchronize()
            assert (room[size:] == 0x5A).all(), (what, size)
            if seen is None:
                seen = out.double()
            err = ((out.double() - seen).norm() / seen.norm()).item()
            # two kernels' fp32 sums; bf16 outputs may differ by a step where they lie across a rounding boundary
            assert err <= (1e-3 if act and op != rn.OP_BWD_WEIGHT else 2e-6), (what, size, need, err)


@pytest.mark.parametrize("plan", [None, "128,128,2", "128,64,1", "64,128,3", "64,64,5"])
@pytest.mark.parametrize("case", [(1, 24, 9, 40, 3, 1, 1), (3, 96, 13, 160, 3, 2, 1), (2, 136, 11, 264, 1, 1, 0), (2, 64, 15, 128, 1, 2, 0)])
def test_filter_gradient_of_bf16_activations(case, plan):
    """Pixel counts that are no multiple of a stage, ragged tiles on both sides, padding and strides.  The products of bf16 operands
    are exact in fp32, the sums round 16 products at a time: the bar of the fp32 filter gradients."""
    n, c, h, k, r, stride, pad = case
    d = _desc(case, True)
    x, w, dy = _operands(case, 9 + sum(case), torch.bfloat16)
    g = torch.Generator().manual_seed(c + k)
    scale, shift = torch.rand(c, generator=g) + 0.5, torch.randn(c, generator=g) * 0.3
    # the BN + ReLU output as stored: one rounding of the fused multiply-add, one to bf16
    z = (x.double() * scale.double() + shift.double()).float().relu().to(torch.bfloat16)
    if plan:
        rn.rn50_set_option("wgrad_plan", plan)
    try:
        ws = ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_WEIGHT))
        dw, dwz, fused = (torch.full(w.shape, 7.0, device="cuda") for _ in range(3))
        rn.conv2d_bwd_weight(d, x.cuda(), dy.cuda(), dw, ws)
        rn.conv2d_bwd_weight(d, z.cuda(), dy.cuda(), dwz, ws)
        rn.conv2d_bwd_weight_bnrelu_input(d, x.cuda(), scale.cuda(), shift.cuda(), dy.cuda(), fused, ws)
        torch.cuda.synchronize()
    finally:
        rn.rn50_set_option("wgrad_plan", None)
    ref = torch.nn.grad.conv2d_weight(_nchw64(x), (k, c, r, r), _nchw64(dy), stride, pad).permute(0, 2, 3, 1)
    assert _err(dw, ref) <= 8e-7
    assert torch.equal(fused, dwz)
