"""The fully connected layer at the edges of its tiles: fewer and more samples, classes and features than a tile, remainders of the
reduction steps, infinite operands.  References: float64 on the CPU."""
import pytest
import torch

from paper_1711_04325_amd import binding as rn

pytestmark = pytest.mark.gpu


def _run(n, j, k, f, w, b, dy):
    y, df, dw, db = (torch.full(s, 7.0, device="cuda") for s in ((n, k), (n, j), (k, j), (k,)))
    rn.fc_fwd(n, j, k, f.cuda(), w.cuda(), b.cuda(), y)
    rn.fc_bwd(n, j, k, f.cuda(), w.cuda(), dy.cuda(), df, dw, db)
    torch.cuda.synchronize()
    return [t.double().cpu() for t in (y, df, dw, db)]


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -120])
@pytest.mark.parametrize("n,j,k", [(1, 4, 1), (3, 36, 17), (16, 2048, 1000), (17, 516, 15), (33, 100, 33), (40, 2052, 21), (65, 64, 1000)])
def test_fully_connected(n, j, k, scale):
    """Sums of exact products rounded 32 at a time (fwd, df) or sample by sample (dw, db: up to 65 of them, 2^-25 * sqrt(65) * 2): below 8e-7.
    With weights and output gradients of 1e-36 as well, whose low bits lie below the smallest bf16 number."""
    g = torch.Generator().manual_seed(n + j + k)
    f, w, b, dy = torch.randn(n, j, generator=g), torch.randn(k, j, generator=g), torch.randn(k, generator=g), torch.randn(n, k, generator=g)
    if scale != 1.0:   # df multiplies two of these: only one of them is small
        ws, bs = w * scale, b * scale
        got = _run(n, j, k, f, ws, bs, dy)
        for what, a, ref in (("y", got[0], f.double() @ ws.double().t() + bs.double()), ("df", got[1], dy.double() @ ws.double())):
            assert ((a - ref).norm() / ref.norm()).item() <= 8e-7, what
        dy = dy * scale
    f64, w64, dy64 = f.double(), w.double(), dy.double()
    refs = (f64 @ w64.t() + b.double(), dy64 @ w64, dy64.t() @ f64, dy64.sum(0))
    for what, got, ref in zip(("y", "df", "dw", "db"), _run(n, j, k, f, w, b, dy), refs):
        assert ((got - ref).norm() / ref.norm()).item() <= 8e-7, what


@pytest.mark.parametrize("n", [1, 32])
def test_operands_of_one_sign(n):
    """Nothing cancels: the sums of the network's last layers to the rounding of their last additions.  A sum added in pairs, pairs of
    pairs, ... has one rounding of its size, two of half of it, four of a quarter: sqrt(1 + 1/2 + 1/4 + ...) < 1.42 roundings of 2.5e-8
    rms, and a little from the short sums at the bottom: below 4.5e-8.  The average of 49 is multiplied by a rounded 1/49 as well (another
    rounding, and up to 3e-8 that all averages share): below 6e-8."""
    g = torch.Generator().manual_seed(n)
    x = torch.randn(n, 7, 7, 2048, generator=g).relu()
    f = torch.full((n, 2048), 7.0, device="cuda")
    rn.avgpool_fwd(n, 2048, 7, 7, x.cuda(), f)
    w, dy, b = torch.rand(1000, 2048, generator=g) * 0.1, torch.rand(n, 1000, generator=g), torch.zeros(1000)
    f = f.cpu()
    y, df, _, _ = _run(n, 2048, 1000, f, w, b, dy)
    for what, got, ref, bar in (("average", f.double(), x.double().mean((1, 2)), 6e-8), ("y", y, f.double() @ w.double().t(), 4.5e-8),
                                ("df", df, dy.double() @ w.double(), 4.5e-8)):
        assert ((got - ref).norm() / ref.norm()).item() <= bar, (what, ((got - ref).norm() / ref.norm()).item())


def test_infinite_operands():
    n, j, k = 20, 68, 37
    g = torch.Generator().manual_seed(4)
    f, w, b, dy = torch.randn(n, j, generator=g), torch.randn(k, j, generator=g), torch.randn(k, generator=g), torch.randn(n, k, generator=g)
    f[3, 67], w[36, 5], dy[19, 2], f[7, 0] = float("inf"), float("-inf"), float("nan"), 3.4e38
    y, df, dw, db = _run(n, j, k, f, w, b, dy)
    f64, w64, dy64 = f.double(), w.double(), dy.double()
    for got, ref in ((y, f64 @ w64.t() + b.double()), (df, dy64 @ w64), (dw, dy64.t() @ f64), (db, dy64.sum(0))):
        ref32 = ref.float().double()  # beyond the fp32 range: infinite
        assert torch.isnan(got[torch.isnan(ref32)]).all()
        assert torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
        fine = torch.isfinite(ref32) & (ref.abs() < 1e30)
        assert ((got - ref)[fine].norm() / ref[fine].norm()).item() <= 8e-7
