"""The first layer's kernels on the bf16 matrix instruction: whole and ragged tiles of 8 x 16 pixels, images of one tile and of many,
split fp32 operands and bf16 activations.  References: float64 on the CPU from the operands as the kernels round them."""
import pytest
import torch

from paper_1711_04325_amd import binding as rn
from tests.gpu_util import ws_bytes

pytestmark = pytest.mark.gpu

# (n, h): 16 x 16 outputs (two tiles), 32 x 32, 19 x 19 (ragged both ways), 9 x 9 (less than a tile wide), more tiles than workgroups
SIZES = [(1, 32), (3, 64), (2, 37), (1, 17), (40, 96)]


def _problem(n, h, act, seed=0):
    g = torch.Generator().manual_seed(n + h + seed)
    p = (h - 1) // 2 + 1
    x, w, dy = torch.randn(n, h, h, 3, generator=g), torch.randn(64, 7, 7, 3, generator=g) * 0.1, torch.randn(n, p, p, 64, generator=g)
    dy = dy.to(torch.bfloat16) if act else dy
    return x, w, dy, rn.conv_desc(n, 3, h, h, 64, 7, 7, 2, 3, in_dtype=rn.DTYPE_BF16_ACT_F32IN if act else rn.DTYPE_F32)


def _refs(x, w, dy, act):
    xq, wq = (x.to(torch.bfloat16), w.to(torch.bfloat16)) if act else (x, w)
    x64, w64, dy64 = (t.double().permute(0, 3, 1, 2) for t in (xq, wq, dy))
    y = torch.nn.functional.conv2d(x64, w64, stride=2, padding=3).permute(0, 2, 3, 1)
    return y, torch.nn.grad.conv2d_weight(x64, w64.shape, dy64, 2, 3).permute(0, 2, 3, 1)


def _run(x, w, dy, d):
    y, dw = torch.full_like(dy, 7.0).cuda(), torch.full_like(w, 7.0).cuda()
    rn.conv2d_fwd(d, x.cuda(), w.cuda(), y, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD)))
    rn.conv2d_bwd_weight(d, x.cuda(), dy.cuda(), dw, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_WEIGHT)))
    torch.cuda.synchronize()
    return y.cpu(), dw.cpu()


@pytest.mark.parametrize("act", [False, True])
@pytest.mark.parametrize("n,h", SIZES)
def test_first_layer(n, h, act):
    """Forward: 147 products, rounded 16 at a time; stored as bf16 off by at most 2^-9 each.  Filter gradient: at most 92,160 pixels in
    512 ranges, six roundings of 2^-25 per 16 pixels of a range (180 pixels), then 512 partial sums: below 1e-6."""
    x, w, dy, d = _problem(n, h, act)
    (y, dw), (y_ref, dw_ref) = _run(x, w, dy, d), _refs(x, w, dy, act)
    err = ((y.double() - y_ref).norm() / y_ref.norm()).item()
    assert err <= (2.0 ** -9 + 1e-5 if act else 8e-7), err
    err = ((dw.double() - dw_ref).norm() / dw_ref.norm()).item()
    assert err <= 1e-6, err


@pytest.mark.parametrize("sx,sw", [(2.0 ** -120, 1.0), (1.0, 2.0 ** -120)])
def test_first_layer_at_the_bottom_of_the_range(sx, sw):
    """Images, or filters and output gradients, of 1e-36: their low bits lie below the smallest bf16 number."""
    x, w, dy, d = _problem(3, 64, False)
    x, w, dy = x * sx, w * sw, dy * sw
    (y, dw), (y_ref, dw_ref) = _run(x, w, dy, d), _refs(x, w, dy, False)
    assert ((y.double() - y_ref).norm() / y_ref.norm()).item() <= 8e-7
    assert ((dw.double() - dw_ref).norm() / dw_ref.norm()).item() <= 1e-6


@pytest.mark.parametrize("act", [False, True])
@pytest.mark.parametrize("n,h", SIZES)
def test_first_layer_statistics(n, h, act):
    """The statistics are those of the output as stored, whichever kernel gathers them; the output is the plain call's."""
    x, w, dy, d = _problem(n, h, act)
    y = torch.full_like(dy, 7.0).cuda()
    gamma, beta = torch.ones(64).cuda(), torch.zeros(64).cuda()
    mean, inv, scale, shift = (torch.empty(64, device="cuda") for _ in range(4))
    rn.conv2d_fwd_bnstats(d, x.cuda(), None, None, w.cuda(), y, gamma, beta, 2e-5, mean, inv, scale, shift,
                          ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_FWD_BNSTATS)))
    torch.cuda.synchronize()
    y64 = y.double().cpu().reshape(-1, 64)
    var = y64.var(0, unbiased=False)
    assert (mean.double().cpu() - y64.mean(0)).abs().max() <= 1e-6 * var.sqrt().max()
    ref = 1.0 / (var + 2e-5).sqrt()
    assert ((inv.double().cpu() - ref).abs() / ref).max() <= 1e-6
    plain, _ = _run(x, w, dy, d)
    err = ((y.double().cpu() - plain.double()).norm() / plain.double().norm()).item()
    assert err <= (1e-3 if act else 1e-7), err   # bf16: a sum across a rounding boundary may go either way


@pytest.mark.parametrize("n,h", [(3, 64), (2, 37)])
def test_first_layer_values_without_a_finite_split(n, h):
    x, w, dy, d = _problem(n, h, False, seed=3)
    x[0, 5, 7, 1], x[n - 1, h - 1, h - 2, 2], x[0, 20, 3, 0], x[1, 9, 9, 0] = float("inf"), float("-inf"), float("nan"), 3.4e38
    (y, dw), (y_ref, dw_ref) = _run(x, w, dy, d), _refs(x, w, dy, False)
    ref32 = y_ref.float()
    assert torch.isnan(y[torch.isnan(ref32)]).all()
    assert torch.equal(y[torch.isinf(y_ref)], ref32[torch.isinf(y_ref)])
    fine = torch.isfinite(ref32) & (y_ref.abs() < 1e30)
    assert torch.isfinite(y[fine]).all() and ((y.double() - y_ref)[fine].norm() / y_ref[fine].norm()).item() <= 8e-7
    # the filter gradient: an infinity of the reference is one of the same sign.  In the ragged tiles of 37 x 37 pixels outside the output
    # multiply the image with zeros, which may make a NaN of it
    got = dw.double()
    assert torch.isnan(got[torch.isnan(dw_ref)]).all()
    inf, fine = torch.isinf(dw_ref), torch.isfinite(dw_ref) & (dw_ref.abs() < 1e30)
    assert ((got[inf] == dw_ref[inf]) | (torch.isnan(got[inf]) & (h == 37))).all()
    assert (torch.isfinite(got[fine]) | (torch.isnan(got[fine]) & (h == 37))).all()


@pytest.mark.parametrize("pixel", [(0, 2, 5), (0, 2, 20), (39, 40, 47)])
def test_first_layer_infinite_output_gradient(pixel):
    """One infinity in one output channel, in the image tile of an even and of an odd workgroup (every other one multiplies with negated
    gradients) and of a workgroup's second tile.  The workgroup forms its sums again on the fp32 instruction: the channel's gradients are
    infinities of the image's signs, all others are what they are without it."""
    n, h = SIZES[-1]
    x, w, dy, d = _problem(n, h, False, seed=5)
    _, clean = _refs(x, w, dy, False)
    dy[pixel][5] = float("inf")
    _, dw = _run(x, w, dy, d)
    im, oh, ow = pixel
    xp = torch.nn.functional.pad(x[im], (0, 0, 3, 3, 3, 3))[2 * oh:2 * oh + 7, 2 * ow:2 * ow + 7]   # what the pixel's filter lies on
    inside = xp != 0.0   # zero padding times an infinity
    assert torch.equal(dw[5][inside], torch.sign(xp[inside]) * float("inf")) and torch.isnan(dw[5][~inside]).all()
    others = [k for k in range(64) if k != 5]
    assert torch.isfinite(dw[others]).all()
    assert ((dw[others].double() - clean[others]).norm() / clean[others].norm()).item() <= 1e-6
