"""The work that a user of librn50 has it do, as cases that can be timed and compared.

A case names one piece of a training or validation iteration of ResNet-50 (its "kind") and its sizes:

  step      one rn50_step of a whole training iteration (forward, loss, backward, fp16 pack, update)
  eval      rn50_forward_eval: validation forward of a whole network, logits out
  unit_fwd  a convolution unit's forward pass: conv2d_fwd_bnstats (optionally with the previous unit's BN + ReLU applied to
            its input as it loads) and bn_fwd_apply
  unit_bwd  the same unit's backward pass: BN + ReLU backward, data gradient, filter gradient
  stem      the first layer's unit with its max pooling, forward and backward
  residual  the BN + residual + ReLU that ends a bottleneck block, forward and backward with the byte mask
  head      average pooling, FC layer and softmax cross-entropy, forward and backward
  update    fp16 gradient pack and the parameter update over flat arenas

dtype: "f32" (the paper's single precision), "bf16" (fp32 tensors, products of operands rounded to bfloat16) or "bf16act"
(activations kept as bfloat16 in memory).
"""
import math

import torch

from paper_1711_04325_amd import binding as rn

DEV = "cuda:0"
EPS = 2e-5
DTYPES = {"f32": rn.DTYPE_F32, "bf16": rn.DTYPE_BF16, "bf16act": rn.DTYPE_BF16_ACT}
PARAMS = 25557032


def listed():
    return [
        # validation of a single image: some 110 dependent launches of small tensors, nothing else in flight
        {"name": "eval_n1", "kind": "eval", "n": 1},
        # the paper's workload: one worker's iteration on its 32 images
        {"name": "step_n32", "kind": "step", "n": 32, "variant": 0, "dtype": "f32"},
        # the largest batch of the sweep, in the variant that keeps activations as bf16
        {"name": "step_n256_bf16act", "kind": "step", "n": 256, "variant": 0, "dtype": "bf16act"},
        # the 3x3 convolution in the middle of a stage-3 block
        {"name": "fwd_3x3_n32_c128_h28", "kind": "unit_fwd", "n": 32, "c": 128, "h": 28, "k": 128, "r": 3, "stride": 1, "dtype": "f32", "fused": False},
        # the widening 1x1 of stage 2 at its full resolution: few products per byte, input normalised as it is read
        {"name": "bwd_1x1_n32_c64_h56_k256", "kind": "unit_bwd", "n": 32, "c": 64, "h": 56, "k": 256, "r": 1, "stride": 1, "dtype": "f32", "fused": True},
        # a long reduction at a large batch
        {"name": "bwd_3x3_n128_c256_h14", "kind": "unit_bwd", "n": 128, "c": 256, "h": 14, "k": 256, "r": 3, "stride": 1, "dtype": "f32", "fused": False},
        # nothing of it fits a tile: odd batch, odd image, strided, widths between the network's
        {"name": "bwd_3x3s2_n9_c96_h29_k160", "kind": "unit_bwd", "n": 9, "c": 96, "h": 29, "k": 160, "r": 3, "stride": 2, "dtype": "f32", "fused": False},
        # narrow activations: the widening 1x1 of stage 4 at a large batch, bound by memory
        {"name": "fwd_1x1_n128_c256_h14_k1024_bf16act", "kind": "unit_fwd", "n": 128, "c": 256, "h": 14, "k": 1024, "r": 1, "stride": 1, "dtype": "bf16act", "fused": False},
        {"name": "bwd_3x3_n64_c128_h28_bf16act", "kind": "unit_bwd", "n": 64, "c": 128, "h": 28, "k": 128, "r": 3, "stride": 1, "dtype": "bf16act", "fused": False},
        # the first layer with its pooling
        {"name": "stem_n32", "kind": "stem", "n": 32, "h": 224},
        # the end of a stage-2 block: five tensors of 103 MB through memory
        {"name": "residual_n32_c256_h56", "kind": "residual", "n": 32, "c": 256, "h": 56},
        # the end of the network: nine small launches
        {"name": "head_n32", "kind": "head", "n": 32},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "eval", "unit_fwd", "unit_fwd", "unit_bwd", "unit_bwd", "stem", "residual", "head", "update"])
    if kind == "step":
        return {"kind": kind, "n": _log(rng, 1, 96), "variant": rng.randrange(2), "dtype": rng.choice(["f32", "f32", "bf16", "bf16act"])}
    if kind == "eval":
        return {"kind": kind, "n": _log(rng, 1, 64)}
    if kind == "stem":
        return {"kind": kind, "n": _log(rng, 1, 64), "h": rng.choice([224, 224, 160, 192, 97, 127])}
    if kind == "residual":
        c, h = rng.choice([(256, 56), (512, 28), (1024, 14), (2048, 7), (64 * rng.randrange(1, 9), rng.randrange(5, 40))])
        return {"kind": kind, "n": _log(rng, 1, 128), "c": c, "h": h}
    if kind == "head":
        return {"kind": kind, "n": _log(rng, 1, 256)}
    if kind == "update":
        return {"kind": kind, "count": _log(rng, 10000, PARAMS)}
    while True:
        r = rng.choice([1, 3])
        width = rng.choice([[64, 128, 256, 512, 1024, 2048], [32 * i for i in range(1, 21)], [8 * i for i in range(2, 30)]])
        c, k = rng.choice(width), rng.choice(width)
        n, h = _log(rng, 1, 128), rng.choice([56, 28, 14, 7, rng.randrange(5, 60)])
        stride = rng.choice([1, 1, 2])
        dtype = rng.choice(["f32", "f32", "f32", "bf16", "bf16act"])
        fused = r == 1 and c % 32 == 0 and rng.random() < 0.3
        p = _out(h, r, stride)
        if 2 * n * p * p * k * c * r * r < 6e11 and n * h * h * max(c, k) < 1.5e8:
            return {"kind": kind, "n": n, "c": c, "h": h, "k": k, "r": r, "stride": stride, "dtype": dtype, "fused": fused}


# ---- shapes ---------------------------------------------------------------------------------------------------------

def _out(h, r, stride):
    return (h + 2 * (r // 2) - r) // stride + 1


def _layers(variant=0):
    """(name, c, k, r, stride, input size) of the 53 convolutions in parameter order."""
    out, cur, c_in = [("stem", 3, 64, 7, 2, 224)], 56, 64
    for stage, (width, blocks) in enumerate([(64, 3), (128, 4), (256, 6), (512, 3)], 2):
        for b in range(blocks):
            down = 2 if b == 0 and stage > 2 else 1
            sa = down if variant == 0 else 1
            name = "s%d.b%d." % (stage, b)
            out.append((name + "a", c_in, width, 1, sa, cur))
            out.append((name + "b", width, width, 3, down // sa, cur // sa))
            out.append((name + "c", width, 4 * width, 1, 1, cur // down))
            if b == 0:
                out.append((name + "p", c_in, 4 * width, 1, down, cur))
            cur, c_in = cur // down, 4 * width
    return out


def work(case):
    kind, n = case["kind"], case.get("n", 0)
    if kind in ("step", "eval"):
        act = 2 if case.get("dtype") == "bf16act" else 4
        macs = elems = 0
        for _, c, k, r, stride, h in _layers(case.get("variant", 0)):
            p = _out(h, r, stride)
            macs += n * p * p * k * c * r * r
            elems += n * p * p * k
        first = n * 112 * 112 * 64 * 147
        image = n * 224 * 224 * 3 * 4
        if kind == "eval":
            return {"flops": 2 * macs, "bytes": image + 4 * PARAMS + 4 * n * 1000}
        # every convolution output has to be kept for the backward pass and read there; state is read and written
        return {"flops": 6 * macs - 2 * first, "bytes": 2 * image + 2 * act * elems + PARAMS * (4 * 3 * 2 + 4 + 2)}
    if kind in ("unit_fwd", "unit_bwd"):
        c, h, k, r = case["c"], case["h"], case["k"], case["r"]
        p = _out(h, r, case["stride"])
        act = 2 if case["dtype"] == "bf16act" else 4
        x, y, w, macs = n * h * h * c, n * p * p * k, k * r * r * c, n * p * p * k * c * r * r
        if kind == "unit_fwd":
            return {"flops": 2 * macs, "bytes": act * (x + 2 * y) + 4 * w}
        return {"flops": 4 * macs, "bytes": act * (2 * x + 3 * y) + 8 * w}
    if kind == "stem":
        p = _out(case["h"], 7, 2)
        q = (p - 1) // 2 + 1
        x, y, z = n * case["h"] ** 2 * 3, n * p * p * 64, n * q * q * 64
        return {"flops": 4 * n * p * p * 64 * 147, "bytes": 4 * x + 3 * 4 * y + 4 * 2 * z + z}
    if kind == "residual":
        e = n * case["c"] * case["h"] ** 2
        return {"flops": 20 * e, "bytes": 4 * 7 * e + e // 4}  # x, residual, y; dy, dy2, dx, dresidual; mask
    if kind == "head":
        return {"flops": 6 * n * 2048 * 1000, "bytes": 4 * (2 * n * 49 * 2048 + 3 * 2048 * 1000 + 2 * n * 1000)}
    return {"flops": 12 * case["count"], "bytes": 30 * case["count"]}


def tolerance(case):
    kind, dtype = case["kind"], case.get("dtype", "f32")
    if kind == "step":
        return TOL_STEP[dtype]
    if kind in ("unit_fwd", "unit_bwd") and dtype == "bf16act":
        return {"rel": 7e-3, "max": 0.03}     # 1.7e-3 (max 7e-3) against 64 bits: a rounding to 8 bits per stored value
    if kind in ("unit_fwd", "unit_bwd") and dtype == "bf16":
        # 1.1e-6 (max 1.2e-4) against 64 bits; a BN-input gradient that falls on the other side of a rounding boundary moves an
        # operand by 2^-8, some 3e-4 of them under another order of the sums before it: 5e-5
        return {"rel": 2e-4, "max": 5e-3}
    if kind == "eval":
        return {"rel": 2e-6, "max": 4e-5}     # 1.3e-7 against 64 bits with one order of the sums
    return {"rel": 8e-6, "max": 4e-4}         # up to 2.1e-6 (max 2.8e-5) against 64 bits: fp32 sums of up to 400,000 terms


# Updated weights after one iteration, the same code with its sums in other orders (other tiles, a separate statistics pass):
# f32 differs by up to 2.5e-4 (max 0.07), because a near tie at a ReLU goes either way and the layers behind it follow; with
# operands or activations of 8 bits by 6e-3 to 9e-3 (max 0.13).
TOL_STEP = {"f32": {"rel": 1e-3, "max": 0.3}, "bf16": {"rel": 0.03, "max": 0.5}, "bf16act": {"rel": 0.03, "max": 0.5}}


# ---- inputs ---------------------------------------------------------------------------------------------------------

class _Draw:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, *shape, std=1.0, mean=0.0):
        return torch.randn(shape, generator=self.g, device=DEV).mul_(std).add_(mean)

    def uniform(self, lo, hi, *shape):
        return torch.rand(shape, generator=self.g, device=DEV).mul_(hi - lo).add_(lo)

    def labels(self, n):
        return torch.randint(0, 1000, (n,), generator=self.g, device=DEV, dtype=torch.int32)

    def theta(self):
        """Flat parameters: He-normal filters, BN scale near 1 and shift near 0, a small FC layer."""
        flat = torch.zeros(rn.rn50_param_count(), device=DEV)
        for _, off, cnt, dims, kind in rn.rn50_param_table():
            part = flat[off:off + cnt]
            if kind == 0:
                part.copy_(self.normal(cnt, std=math.sqrt(2.0 / (dims[1] * dims[2] * dims[3]))))
            elif kind == 1:
                part.copy_(self.normal(cnt, std=0.1, mean=1.0))
            elif kind == 2:
                part.copy_(self.normal(cnt, std=0.1))
            elif kind == 3:
                part.copy_(self.normal(cnt, std=0.01))
        return flat


def _empty(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _ws(nbytes):
    return _empty(max(16, int(nbytes)), dtype=torch.uint8)


def _channel_stats(y):
    """Mean and 1/sigma per channel of an NHWC tensor, as the forward pass saved them."""
    f = y.reshape(-1, y.shape[-1]).double()
    mean = f.mean(0)
    return mean.float(), (1.0 / torch.sqrt((f - mean).square().mean(0) + EPS)).float()


def prepare(case, seed):
    with torch.no_grad():
        s = _PREPARE[case["kind"]](case, _Draw(seed))
    s["case"] = case
    return s


def _prepare_step(case, g):
    n = case["n"]
    s = {"images": g.normal(n, 224, 224, 3), "labels": g.labels(n), "theta": g.theta()}
    s["ctx"] = rn.Rn50Ctx(n, variant=case["variant"], conv_dtype=DTYPES[case["dtype"]])
    # a state some iterations into the warm-up: momentum and second moments of gradient-sized values
    s["delta"], s["m"] = g.normal(rn.rn50_param_count(), std=1e-3), g.uniform(1e-6, 1e-4, rn.rn50_param_count())
    s["grad"], s["grad16"], s["loss"] = torch.empty_like(s["theta"]), _empty(s["theta"].numel(), dtype=torch.int16), _empty(1)
    s["hp"] = rn.rn50_recipe_hparams(2.0, 1, n)
    return s


def _prepare_eval(case, g):
    n = case["n"]
    s = {"images": g.normal(n, 224, 224, 3), "theta": g.theta(), "logits": _empty(n, 1000), "ctx": rn.Rn50Ctx(n), "stats": []}
    for i, (_, _, k, _, _, _) in enumerate(_layers()):
        mean, invstd = g.normal(k, std=0.1), g.uniform(0.4, 0.7, k)
        s["ctx"].set_bn_stats(i, mean, invstd)
        s["stats"].append((mean, invstd))
    return s


def _unit(case, g):
    n, c, h, k, r, stride = (case[f] for f in ("n", "c", "h", "k", "r", "stride"))
    p = _out(h, r, stride)
    act = torch.bfloat16 if case["dtype"] == "bf16act" else torch.float32
    s = {"desc": rn.conv_desc(n, c, h, h, k, r, r, stride, r // 2, in_dtype=DTYPES[case["dtype"]]), "p": p, "act": act}
    # the input of a unit: the ReLU output of the one before, or what that one's BN + ReLU will be applied to
    x = g.normal(n, h, h, c)
    s["x"] = (x if case["fused"] else x.relu_()).to(act)
    s["scale_in"], s["shift_in"] = (g.uniform(0.5, 1.5, c), g.normal(c, std=0.3)) if case["fused"] else (None, None)
    s["w"] = g.normal(k, r, r, c, std=math.sqrt(2.0 / (c * r * r)))
    s["gamma"], s["beta"] = g.normal(k, std=0.1, mean=1.0), g.normal(k, std=0.1)
    return s


def _prepare_unit_fwd(case, g):
    s = _unit(case, g)
    n, k, p = case["n"], case["k"], s["p"]
    s["y"], s["z"] = _empty(n, p, p, k, dtype=s["act"]), _empty(n, p, p, k, dtype=s["act"])
    s["mean"], s["invstd"], s["scale"], s["shift"] = (_empty(k) for _ in range(4))
    s["ws"] = _ws(rn.rn50_conv_workspace_bytes(s["desc"], rn.OP_FWD_BNSTATS))
    return s


def _prepare_unit_bwd(case, g):
    s = _unit(case, g)
    n, c, h, k, r, p = case["n"], case["c"], case["h"], case["k"], case["r"], s["p"]
    s["y"] = (g.normal(n, p, p, k) * g.uniform(0.8, 1.6, k) + g.normal(k, std=0.5)).to(s["act"])
    s["mean"], s["invstd"] = _channel_stats(s["y"])
    s["dz"] = g.normal(n, p, p, k, std=0.01).to(s["act"])
    s["dy"], s["dx"], s["dw"] = torch.empty_like(s["y"]), torch.empty_like(s["x"]), torch.empty_like(s["w"])
    s["dgamma"], s["dbeta"] = _empty(k), _empty(k)
    s["ws_bn"] = _ws(rn.rn50_bn_workspace_bytes(n, k, p, p))
    s["ws_d"] = _ws(rn.rn50_conv_workspace_bytes(s["desc"], rn.OP_BWD_DATA))
    s["ws_w"] = _ws(rn.rn50_conv_workspace_bytes(s["desc"], rn.OP_BWD_WEIGHT))
    return s


def _prepare_stem(case, g):
    n, h = case["n"], case["h"]
    p = _out(h, 7, 2)
    q = (p - 1) // 2 + 1
    s = {"desc": rn.conv_desc(n, 3, h, h, 64, 7, 7, 2, 3), "p": p, "x": g.normal(n, h, h, 3), "w": g.normal(64, 7, 7, 3, std=math.sqrt(2.0 / 147))}
    s["gamma"], s["beta"] = g.normal(64, std=0.1, mean=1.0), g.normal(64, std=0.1)
    s["y"], s["pool"], s["arg"] = _empty(n, p, p, 64), _empty(n, q, q, 64), _empty(n, q, q, 64, dtype=torch.uint8)
    # pooling and backward pass start from a convolution output of their own: a near tie that another rounding of the
    # convolution turns would move a whole gradient to another pixel
    s["saved"] = g.normal(n, p, p, 64) * g.uniform(0.8, 1.6, 64) + g.normal(64, std=0.5)
    s["saved_mean"], s["saved_invstd"] = _channel_stats(s["saved"])
    scale, shift = _affine(s["gamma"], s["beta"], s["saved_mean"], s["saved_invstd"])
    s["saved_scale"], s["saved_shift"] = scale.float(), shift.float()
    s["dpool"] = g.normal(n, q, q, 64, std=0.01)
    s["dz"], s["dy"], s["dw"] = _empty(n, p, p, 64), _empty(n, p, p, 64), torch.empty_like(s["w"])
    s["mean"], s["invstd"], s["scale"], s["shift"], s["dgamma"], s["dbeta"] = (_empty(64) for _ in range(6))
    s["ws_f"] = _ws(rn.rn50_conv_workspace_bytes(s["desc"], rn.OP_FWD_BNSTATS))
    s["ws_w"] = _ws(rn.rn50_conv_workspace_bytes(s["desc"], rn.OP_BWD_WEIGHT))
    s["ws_bn"] = _ws(rn.rn50_bn_workspace_bytes(n, 64, p, p))
    return s


def _prepare_residual(case, g):
    n, c, h = case["n"], case["c"], case["h"]
    shape = (n, h, h, c)
    s = {"x": g.normal(*shape) * g.uniform(0.8, 1.6, c) + g.normal(c, std=0.5), "res": g.normal(*shape).relu_()}
    s["gamma"], s["beta"] = g.normal(c, std=0.1, mean=1.0), g.normal(c, std=0.1)
    s["dz"], s["dz2"] = g.normal(*shape, std=0.01), g.normal(*shape, std=0.01)
    s["z"], s["dx"], s["dres"], s["mask"] = _empty(*shape), _empty(*shape), _empty(*shape), _empty(n * h * h * c // 4, dtype=torch.uint8)
    s["mean"], s["invstd"], s["dgamma"], s["dbeta"] = (_empty(c) for _ in range(4))
    s["ws"] = _ws(rn.rn50_bn_workspace_bytes(n, c, h, h))
    return s


def _prepare_head(case, g):
    n = case["n"]
    s = {"x": g.normal(n, 7, 7, 2048).relu_(), "w": g.normal(1000, 2048, std=0.01), "b": g.normal(1000, std=0.01), "labels": g.labels(n)}
    s["f"], s["logits"], s["loss"], s["dlogits"] = _empty(n, 2048), _empty(n, 1000), _empty(1), _empty(n, 1000)
    s["df"], s["dw"], s["db"], s["dx"] = _empty(n, 2048), _empty(1000, 2048), _empty(1000), _empty(n, 7, 7, 2048)
    return s


def _prepare_update(case, g):
    cnt = case["count"]
    s = {"theta": g.normal(cnt, std=0.05), "delta": g.normal(cnt, std=1e-3), "m": g.uniform(1e-6, 1e-4, cnt)}
    s["g"] = g.normal(cnt) * torch.exp(g.uniform(math.log(1e-6), 0.0, cnt))
    s["g16"] = _empty(cnt, dtype=torch.int16)
    s["mask"] = (g.uniform(0.0, 1.0, (cnt + rn.WD_GROUP - 1) // rn.WD_GROUP) < 0.9).to(torch.uint8)
    s["hp"] = rn.rn50_recipe_hparams(8.0, 1024, 32)
    return s


_PREPARE = {"step": _prepare_step, "eval": _prepare_eval, "unit_fwd": _prepare_unit_fwd, "unit_bwd": _prepare_unit_bwd, "stem": _prepare_stem,
            "residual": _prepare_residual, "head": _prepare_head, "update": _prepare_update}


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(s):
    return _RUN[s["case"]["kind"]](s, s["case"])


def _run_step(s, case):
    s["ctx"].step(s["images"], s["labels"], s["theta"], s["grad"], s["delta"], s["m"], s["grad16"], s["hp"], EPS, s["loss"])
    return {"loss": s["loss"], "theta": s["theta"]}


def _run_eval(s, case):
    s["ctx"].forward_eval(s["images"], s["theta"], s["logits"])
    return {"logits": s["logits"]}


def _run_unit_fwd(s, case):
    n, k, p = case["n"], case["k"], s["p"]
    rn.conv2d_fwd_bnstats(s["desc"], s["x"], s["scale_in"], s["shift_in"], s["w"], s["y"], s["gamma"], s["beta"], EPS, s["mean"], s["invstd"],
                          s["scale"], s["shift"], s["ws"])
    apply = rn.bn_fwd_apply_bf16 if case["dtype"] == "bf16act" else rn.bn_fwd_apply
    apply(n, k, p, p, s["y"], s["scale"], s["shift"], None, 1, s["z"])
    return {"y": s["y"], "z": s["z"], "mean": s["mean"], "invstd": s["invstd"]}


def _run_unit_bwd(s, case):
    n, k, p = case["n"], case["k"], s["p"]
    if case["dtype"] == "bf16act":
        rn.bn_bwd_batchstats_bf16(n, k, p, p, s["y"], s["dz"], None, None, None, s["gamma"], s["beta"], s["mean"], s["invstd"], 1, s["dy"], None,
                                  s["dgamma"], s["dbeta"], s["ws_bn"])
    else:
        rn.bn_bwd_batchstats_xmask(n, k, p, p, s["y"], s["dz"], s["gamma"], s["beta"], s["mean"], s["invstd"], s["dy"], s["dgamma"], s["dbeta"],
                                   s["ws_bn"])
    rn.conv2d_bwd_data(s["desc"], s["dy"], s["w"], s["dx"], s["ws_d"])
    if case["fused"]:
        rn.conv2d_bwd_weight_bnrelu_input(s["desc"], s["x"], s["scale_in"], s["shift_in"], s["dy"], s["dw"], s["ws_w"])
    else:
        rn.conv2d_bwd_weight(s["desc"], s["x"], s["dy"], s["dw"], s["ws_w"])
    return {"dy": s["dy"], "dx": s["dx"], "dw": s["dw"], "dgamma": s["dgamma"], "dbeta": s["dbeta"]}


def _run_stem(s, case):
    n, p = case["n"], s["p"]
    rn.conv2d_fwd_bnstats(s["desc"], s["x"], None, None, s["w"], s["y"], s["gamma"], s["beta"], EPS, s["mean"], s["invstd"], s["scale"], s["shift"],
                          s["ws_f"])
    rn.maxpool3x3s2_fwd_bnrelu_input(n, 64, p, p, s["saved"], s["saved_scale"], s["saved_shift"], s["pool"], s["arg"])
    rn.maxpool3x3s2_bwd(n, 64, p, p, s["dpool"], None, s["arg"], s["dz"])
    rn.bn_bwd_batchstats_xmask(n, 64, p, p, s["saved"], s["dz"], s["gamma"], s["beta"], s["saved_mean"], s["saved_invstd"], s["dy"], s["dgamma"],
                               s["dbeta"], s["ws_bn"])
    rn.conv2d_bwd_weight(s["desc"], s["x"], s["dy"], s["dw"], s["ws_w"])
    return {"y": s["y"], "mean": s["mean"], "invstd": s["invstd"], "pool": s["pool"], "arg": s["arg"], "dz": s["dz"], "dy": s["dy"], "dw": s["dw"],
            "dgamma": s["dgamma"], "dbeta": s["dbeta"]}


def _run_residual(s, case):
    n, c, h = case["n"], case["c"], case["h"]
    rn.bn_fwd_batchstats_mask(n, c, h, h, s["x"], s["gamma"], s["beta"], EPS, s["res"], s["z"], s["mask"], s["mean"], s["invstd"], s["ws"])
    rn.bn_bwd_batchstats_mask(n, c, h, h, s["x"], s["dz"], s["dz2"], s["mask"], s["gamma"], s["mean"], s["invstd"], s["dx"], s["dres"], s["dgamma"],
                              s["dbeta"], s["ws"])
    return {"z": s["z"], "mean": s["mean"], "invstd": s["invstd"], "dx": s["dx"], "dres": s["dres"], "dgamma": s["dgamma"], "dbeta": s["dbeta"]}


def _run_head(s, case):
    n = case["n"]
    rn.avgpool_fwd(n, 2048, 7, 7, s["x"], s["f"])
    rn.fc_fwd(n, 2048, 1000, s["f"], s["w"], s["b"], s["logits"])
    rn.softmax_ce(n, 1000, s["logits"], s["labels"], s["loss"], s["dlogits"])
    rn.fc_bwd(n, 2048, 1000, s["f"], s["w"], s["dlogits"], s["df"], s["dw"], s["db"])
    rn.avgpool_bwd(n, 2048, 7, 7, s["df"], s["dx"])
    return {f: s[f] for f in ("f", "logits", "loss", "dlogits", "df", "dw", "db", "dx")}


def _run_update(s, case):
    rn.grad_pack_fp16(case["count"], s["g"], s["g16"])
    rn.opt_update(case["count"], s["theta"], s["delta"], s["m"], None, s["g16"], s["mask"], s["hp"])
    return {"g16": s["g16"], "theta": s["theta"], "delta": s["delta"], "m": s["m"]}


_RUN = {"step": _run_step, "eval": _run_eval, "unit_fwd": _run_unit_fwd, "unit_bwd": _run_unit_bwd, "stem": _run_stem,
        "residual": _run_residual, "head": _run_head, "update": _run_update}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

def exact(case, seed):
    if case["kind"] not in _EXACT:
        return None   # a training step decides millions of ReLUs: near ties turn with any rounding
    with torch.no_grad():
        return _EXACT[case["kind"]](prepare(case, seed), case)


def _taps(x, r, stride, p):
    """For each filter tap (i, j): the input elements it meets, as a [pixels, channels] matrix."""
    pad = r // 2
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    for i in range(r):
        for j in range(r):
            yield i, j, xp[:, i:i + stride * (p - 1) + 1:stride, j:j + stride * (p - 1) + 1:stride, :]


def _conv(x, w, stride):
    k, r = w.shape[0], w.shape[1]
    p = _out(x.shape[1], r, stride)
    y = torch.zeros(x.shape[0] * p * p, k, dtype=torch.float64, device=x.device)
    for i, j, t in _taps(x, r, stride, p):
        y += t.reshape(-1, x.shape[3]) @ w[:, i, j, :].t().contiguous()
    return y.reshape(x.shape[0], p, p, k)


def _conv_dw(x, dy, r, stride):
    p, k = dy.shape[1], dy.shape[3]
    dw = torch.zeros(k, r, r, x.shape[3], dtype=torch.float64, device=x.device)
    flat = dy.reshape(-1, k).t().contiguous()
    for i, j, t in _taps(x, r, stride, p):
        dw[:, i, j, :] = flat @ t.reshape(-1, x.shape[3])
    return dw


def _conv_dx(dy, w, stride, h):
    n, p, _, k = dy.shape
    r, c = w.shape[1], w.shape[3]
    pad = r // 2
    full = torch.zeros(n, h + 2 * pad, h + 2 * pad, c, dtype=torch.float64, device=dy.device)
    flat = dy.reshape(-1, k)
    for i in range(r):
        for j in range(r):
            full[:, i:i + stride * (p - 1) + 1:stride, j:j + stride * (p - 1) + 1:stride, :] += (flat @ w[:, i, j, :].contiguous()).reshape(n, p, p, c)
    return full[:, pad:pad + h, pad:pad + h, :].contiguous()


def _bn_stats(y):
    f = y.reshape(-1, y.shape[-1])
    mean = f.mean(0)
    return mean, 1.0 / torch.sqrt((f - mean).square().mean(0) + EPS)


def _bn_bwd(y, dz, gamma, mean, invstd):
    xhat = (y - mean) * invstd
    dbeta, dgamma = dz.reshape(-1, dz.shape[-1]).sum(0), (dz * xhat).reshape(-1, dz.shape[-1]).sum(0)
    m = dz.numel() / dz.shape[-1]
    return gamma * invstd * (dz - dbeta / m - xhat * dgamma / m), dgamma, dbeta


def _affine(gamma, beta, mean, invstd):
    """Scale and shift of a BN as fp32 numbers (the ReLU's decision is a function of these)."""
    scale = gamma * invstd
    return scale.double(), (beta.double() - mean.double() * scale.double()).float().double()


def _bf16(t, case):
    return t.float().bfloat16().double() if case["dtype"] != "f32" else t


def _unit_input(s, case):
    x = s["x"].double()
    if case["fused"]:
        x = (x * s["scale_in"].double() + s["shift_in"].double()).float().double().relu()
    return _bf16(x, case)   # operands of a bf16 product are the rounded values


def _exact_unit_fwd(s, case):
    y = _conv(_unit_input(s, case), _bf16(s["w"].double(), case), case["stride"])
    seen = y.float().bfloat16().double() if case["dtype"] == "bf16act" else y   # statistics are those of the tensor as stored
    mean, invstd = _bn_stats(seen)
    z = ((seen - mean) * invstd * s["gamma"].double() + s["beta"].double()).relu()
    return {"y": y, "z": z, "mean": mean, "invstd": invstd}


def _exact_unit_bwd(s, case):
    y = s["y"].double()
    scale, shift = _affine(s["gamma"], s["beta"], s["mean"], s["invstd"])
    dz = s["dz"].double() * ((y * scale + shift) > 0)
    dy, dgamma, dbeta = _bn_bwd(y, dz, s["gamma"].double(), s["mean"].double(), s["invstd"].double())
    seen, w, x = _bf16(dy, case), _bf16(s["w"].double(), case), _unit_input(s, case)
    return {"dy": dy, "dx": _conv_dx(seen, w, case["stride"], case["h"]), "dw": _conv_dw(x, seen, case["r"], case["stride"]), "dgamma": dgamma,
            "dbeta": dbeta}


def _exact_stem(s, case):
    x = s["x"].double()
    xp = torch.nn.functional.pad(x, (0, 0, 3, 3, 3, 3))
    n, p = case["n"], s["p"]
    cols = [xp[:, i:i + 2 * (p - 1) + 1:2, j:j + 2 * (p - 1) + 1:2, :] for i in range(7) for j in range(7)]
    cols = torch.cat(cols, 3).reshape(n * p * p, 147)
    y = (cols @ s["w"].double().reshape(64, 147).t().contiguous()).reshape(n, p, p, 64)
    mean, invstd = _bn_stats(y)
    saved = s["saved"].double()
    z = (saved * s["saved_scale"].double() + s["saved_shift"].double()).float().double().relu()   # ties are those of fp32 values
    pool, where = torch.nn.functional.max_pool2d(z.permute(0, 3, 1, 2).contiguous(), 3, 2, 1, return_indices=True)
    dz = torch.zeros(n, 64, p * p, dtype=torch.float64, device=x.device)
    dz.scatter_add_(2, where.reshape(n, 64, -1), s["dpool"].double().permute(0, 3, 1, 2).reshape(n, 64, -1))
    dz = dz.reshape(n, 64, p, p).permute(0, 2, 3, 1).contiguous()
    dy, dgamma, dbeta = _bn_bwd(saved, dz * (z > 0), s["gamma"].double(), s["saved_mean"].double(), s["saved_invstd"].double())
    dw = (dy.reshape(-1, 64).t().contiguous() @ cols).reshape(64, 7, 7, 3)
    return {"y": y, "mean": mean, "invstd": invstd, "pool": pool.permute(0, 2, 3, 1).contiguous(), "arg": None, "dz": dz, "dy": dy, "dw": dw,
            "dgamma": dgamma, "dbeta": dbeta}


def _exact_residual(s, case):
    x, gamma = s["x"].double(), s["gamma"].double()
    mean, invstd = _bn_stats(x)
    z = ((x - mean) * invstd * gamma + s["beta"].double() + s["res"].double()).relu()
    dres = (s["dz"].double() + s["dz2"].double()) * (z > 0)
    dx, dgamma, dbeta = _bn_bwd(x, dres, gamma, mean, invstd)
    return {"z": z, "mean": mean, "invstd": invstd, "dx": dx, "dres": dres, "dgamma": dgamma, "dbeta": dbeta}


def _exact_head(s, case):
    n = case["n"]
    f, w = s["x"].double().mean((1, 2)), s["w"].double()
    logits = f @ w.t().contiguous() + s["b"].double()
    logp = torch.log_softmax(logits, 1)
    hot = torch.nn.functional.one_hot(s["labels"].long(), 1000).double()
    loss, dlogits = -(logp * hot).sum() / n, (logp.exp() - hot) / n
    df = dlogits @ w
    dx = (df / 49).reshape(n, 1, 1, 2048).expand(n, 7, 7, 2048).contiguous()
    return {"f": f, "logits": logits, "loss": loss.reshape(1), "dlogits": dlogits, "df": df, "dw": dlogits.t().contiguous() @ f, "db": dlogits.sum(0),
            "dx": dx}


def _exact_update(s, case):
    hp, theta = s["hp"], s["theta"].double()
    decay = s["mask"].repeat_interleave(rn.WD_GROUP)[:case["count"]].double()
    g = s["g"].half().double() * hp.g_scale + hp.wd * theta * decay
    m = hp.mu2 * s["m"].double() + (1.0 - hp.mu2) * g * g
    delta = hp.mu1 * s["delta"].double() - (hp.a_sgd + hp.a_rms / (m.sqrt() + hp.eps)) * g
    return {"g16": None, "theta": theta + hp.eta * delta, "delta": delta, "m": m}


def _exact_eval(s, case):
    flat, at, layer = s["theta"].double(), [0], [0]

    def take(count):
        at[0] += count
        return flat[at[0] - count:at[0]]

    def unit(x, c, k, r, stride):
        w, gamma, beta = take(k * r * r * c).reshape(k, r, r, c), take(k), take(k)
        mean, invstd = (t.double() for t in s["stats"][layer[0]])
        layer[0] += 1
        return (_conv(x, w, stride) - mean) * invstd * gamma + beta

    layers = _layers()
    x = unit(s["images"].double(), 3, 64, 7, 2).relu()
    x = torch.nn.functional.max_pool2d(x.permute(0, 3, 1, 2).contiguous(), 3, 2, 1).permute(0, 2, 3, 1).contiguous()
    i = 1
    while i < len(layers):
        t, block_in = x, x
        for j in range(3):
            _, c, k, r, stride, _ = layers[i + j]
            t = unit(t, c, k, r, stride)
            t = t.relu() if j < 2 else t
        i += 3
        if i < len(layers) and layers[i][0].endswith(".p"):
            _, c, k, r, stride, _ = layers[i]
            block_in = unit(x, c, k, r, stride)
            i += 1
        x = (t + block_in).relu()
    w, b = take(2048 * 1000).reshape(1000, 2048), take(1000)
    return {"logits": x.mean((1, 2)) @ w.t().contiguous() + b}


_EXACT = {"eval": _exact_eval, "unit_fwd": _exact_unit_fwd, "unit_bwd": _exact_unit_bwd, "stem": _exact_stem, "residual": _exact_residual,
          "head": _exact_head, "update": _exact_update}
