"""Options that change while the library is in use: a call decides everything by the snapshot it started with."""
import threading

import pytest
import torch

from paper_1711_04325_amd import binding as rn
from tests.gpu_util import ws_bytes
from tests.step_util import gpu_forward_backward, problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case,option,value", [((2, 64, 14, 64, 3, 1), "igemm_plan", "64,64,1"), ((2, 128, 8, 64, 1, 2), "igemm_plan", "64,64,1"),
                                               ((5, 160, 6, 224, 3, 1), "operand_plans", "1,5,160,6,224,3,1,1,64,64,1")])
def test_options_set_by_another_thread_during_data_gradients(case, option, value):
    """One setting's kernel reads the filter as it is, the other's a flipped one: a call that asks twice and is told differently takes one for the
    other, and its result is of another filter altogether.  Relative error against 64 bits: see the bars of test_gpu_conv_operands."""
    n, c, h, k, r, stride = case
    g = torch.Generator().manual_seed(sum(case))
    p = (h + 2 * (r // 2) - r) // stride + 1
    dy, w = torch.randn(n, p, p, k, generator=g), torch.randn(k, r, r, c, generator=g) * (2.0 / (c * r * r)) ** 0.5
    ref = torch.nn.grad.conv2d_input((n, c, h, h), w.double().permute(0, 3, 1, 2), dy.double().permute(0, 3, 1, 2), stride, r // 2).permute(0, 2, 3, 1)
    ref = ref.contiguous().cuda()
    d = rn.conv_desc(n, c, h, h, k, r, r, stride, r // 2)
    dy, w, dx, ws = dy.cuda(), w.cuda(), torch.empty(n, h, h, c, device="cuda"), ws_bytes(16 << 20)   # room for either
    stop = threading.Event()

    def toggle():
        while not stop.is_set():
            rn.rn50_set_option(option, value)
            rn.rn50_set_option(option, None)

    other = threading.Thread(target=toggle)
    other.start()
    worst = torch.zeros((), dtype=torch.float64, device="cuda")
    try:
        for _ in range(2000):
            rn.conv2d_bwd_data(d, dy, w, dx, ws)
            worst = torch.maximum(worst, (dx.double() - ref).norm() / ref.norm())
        worst = worst.item()
    finally:
        stop.set()
        other.join()
        rn.rn50_set_option(option, None)
    assert worst <= 8e-7, worst


def test_halves_planned_after_a_context_prepared_its_filters():
    """A context prepares filters as bf16 terms where the options at its creation plan them; a step whose options plan fp16 halves for such a layer
    prepares its own operands (there is no gathered tensor's halves among what the context prepared)."""
    batch = 8
    images, params, labels = problem(31, batch)
    ctx = rn.Rn50Ctx(batch)
    loss, before, theta, dimg, dlab = gpu_forward_backward(ctx, images, params, labels, 2e-5)
    after, again, out = torch.empty_like(before), torch.empty_like(before), torch.empty(1, device="cuda")
    rows = [(256, 56, 64, 1, 1), (64, 56, 64, 3, 1), (128, 28, 128, 3, 1), (512, 28, 128, 1, 1), (256, 14, 256, 3, 1), (1024, 14, 256, 1, 1)]
    rn.rn50_set_option("operand_plans", ";".join("%d,%d,%d,%d,%d,%d,%d,%d,64,64,1" % (rn.OP_BWD_DATA, batch, c, h, k, r, s, r // 2) for c, h, k, r, s in rows))
    try:
        ctx.forward_backward(dimg, dlab, theta, after, 2e-5, out)
        torch.cuda.synchronize()
    finally:
        rn.rn50_set_option("operand_plans", None)
    ctx.forward_backward(dimg, dlab, theta, again, 2e-5, out)
    torch.cuda.synchronize()
    ctx.close()
    assert out.item() == loss and torch.equal(again.view(torch.int32), before.view(torch.int32))
    assert not torch.equal(after.view(torch.int32), before.view(torch.int32))   # the halves ran
    # the forward pass is the same bits, so every ReLU decides alike and what differs are roundings of 1e-7 in the data gradients: as between two
    # orders of the sums in test_gpu_step_group
    for name, off, cnt, dims, kind in rn.rn50_param_table():
        a, b = after[off:off + cnt].double(), before[off:off + cnt].double()
        assert ((a - b).norm() / b.norm().clamp_min(1e-30)).item() <= 1e-5, name
