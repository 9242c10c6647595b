"""GPU parity of strided data gradients whose image has odd sizes: rows of the output are ordered by the parity class of their pixel, and the
classes differ in their number of rows (one may be empty).  Against a sum over filter taps in 64 bits."""
import pytest
import torch

from paper_1711_04325_amd import binding as rn
from tests.gpu_util import DEV, ws_bytes

pytestmark = pytest.mark.gpu

# n, c, h, w, k, r
CASES = [
    (9, 96, 29, 29, 160, 3),     # tiles that straddle classes, pieces of tiles
    (4096, 64, 5, 1, 64, 3),     # no odd columns
    (4096, 64, 1, 7, 64, 3),     # no odd rows
    (16, 96, 21, 23, 64, 5),
    (33, 256, 29, 29, 256, 3),   # large enough for the kernels with a prepared filter
    (80, 512, 15, 13, 512, 3),
    (24, 256, 28, 27, 192, 3),   # odd in one direction only
    (24, 256, 27, 28, 192, 3),
    (2, 32, 7, 7, 64, 3),        # small ones, filters of one tap: in image order
    (3, 36, 8, 7, 32, 3),
    (2, 32, 1, 1, 32, 1),
    (4, 64, 15, 15, 128, 1),
]


@pytest.mark.parametrize("dtype", [rn.DTYPE_F32, rn.DTYPE_BF16, rn.DTYPE_BF16_ACT], ids=["f32", "bf16", "bf16act"])
@pytest.mark.parametrize("case", CASES)
def test_strided_data_gradient_of_an_odd_image(case, dtype):
    n, c, h, w, k, r = case
    if dtype == rn.DTYPE_BF16_ACT and (c % 8 or k % 8):
        pytest.skip("channels of bf16 activations come in eights")
    pad = r // 2
    p, q = (h + 2 * pad - r) // 2 + 1, (w + 2 * pad - r) // 2 + 1
    g = torch.Generator(device=DEV)
    g.manual_seed(sum(case))
    act = torch.bfloat16 if dtype == rn.DTYPE_BF16_ACT else torch.float32
    dy = torch.randn(n, p, q, k, generator=g, device=DEV).to(act)
    wt = torch.randn(k, r, r, c, generator=g, device=DEV)
    dx = torch.full((n, h, w, c), 7.0, device=DEV, dtype=act)   # every element is written
    d = rn.conv_desc(n, c, h, w, k, r, r, 2, pad, in_dtype=dtype)
    rn.conv2d_bwd_data(d, dy, wt, dx, ws_bytes(rn.rn50_conv_workspace_bytes(d, rn.OP_BWD_DATA)))
    dy64, w64 = dy.double(), wt.double()
    if dtype != rn.DTYPE_F32:
        dy64, w64 = dy.float().bfloat16().double(), wt.bfloat16().double()
    full = torch.zeros(n, h + 2 * pad, w + 2 * pad, c, dtype=torch.float64, device=DEV)
    for i in range(r):
        for j in range(r):
            full[:, i:i + 2 * p - 1:2, j:j + 2 * q - 1:2, :] += (dy64.reshape(-1, k) @ w64[:, i, j, :].contiguous()).reshape(n, p, q, c)
    ref = full[:, pad:pad + h, pad:pad + w, :]
    # products of unit normal numbers: a result and its partial sums are of the size of (r*r*k)^0.5, at most 6 of those, and each of its
    # fewer than r*r*k roundings adds 2^-24 of that at the most, some (r*r*k)^0.5 of them together; as bf16, a rounding to 8 bits more
    terms = r * r * k
    err = (dx.double() - ref).abs()
    bound = 6 * terms ** 0.5 * 2.0 ** -24 * 6 * terms ** 0.5
    assert (err <= bound + (2.0 ** -8 * ref.abs() if dtype == rn.DTYPE_BF16_ACT else 0.0)).all()
