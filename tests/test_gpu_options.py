"""Options that change while the library is in use: a call decides everything by the snapshot it started with."""
import threading

import pytest
import torch

from paper_1711_04325_amd import binding as rn
from tests.gpu_util import ws_bytes

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
