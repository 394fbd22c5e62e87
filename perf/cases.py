"""What is timed: the training step of DSP on whole networks, on one block and on one layer.

Three kinds of case, each through the package's public entry points:

  pipeline  a network split into K blocks that trains under its own DSP(p; m) schedule: ``ticks`` calls of
            ``dsp_pipeline_step`` (one fresh mini-batch each: forward, recompute, backward and update in every block),
            the last of which asks for its loss, then the weights are read back -- what a training program does between
            two points at which it reports and saves.  The pipeline is full before the first pass.
  block     one mid-network block driven by its owner on one stream (``dsp_block_step`` or the separate calls, then
            ``dsp_param_update``) with activations from below and an error gradient from above: ``ticks`` steps, then
            the weights are read back.
  layer     one convolution and one batch norm (+ residual) + ReLU, forward and backward, through the single-layer entry
            points, on tensors the caller owns (each call on tensors of its own, as the layers of a network find them).

Sizes are those of the workloads the package is configured for, plus ragged ones of the same ranges.
"""
import math

import numpy as np
import torch

import paper_1909_02625_amd as D
from paper_1909_02625_amd.marshal import block_shapes, build_gpu_blocks, destroy_blocks
from workloads import get_config
from workloads.configs import infer_shapes, param_shapes

_BATCHES = 4          # mini-batches that are resident and taken in turn
_MAX_TICKS = 1 << 22  # loss history of a pipeline
# The step size behind the first drop of a schedule, and the scale a mean loss leaves in the error gradient of a
# mid-network map: at the step size of the first epoch two runs that differ by one rounding part within a few steps.
_LR, _GRAD_STD = 1e-4, 1e-5


def listed():
    return [
        # the smallest network, batch 8: a tick is a few dozen launches of a few microseconds each
        {"name": "tiny2_fp32", "kind": "pipeline", "net": "tiny2", "dtype": "fp32", "batch": 8, "hw": 16, "ticks": 16},
        # CIFAR ResNet-20, K = 3, fp32
        {"name": "resnet20_fp32", "kind": "pipeline", "net": "resnet20", "dtype": "fp32", "batch": 128, "hw": 32, "ticks": 16},
        # CIFAR ResNet-56, K = 4, bf16
        {"name": "resnet56_bf16", "kind": "pipeline", "net": "resnet56", "dtype": "bf16", "batch": 128, "hw": 32, "ticks": 16},
        # the pre-activation bottleneck network of the straggler experiments, K = 3: a thousand small layers
        {"name": "resnet164_fp32", "kind": "pipeline", "net": "resnet164", "dtype": "fp32", "batch": 128, "hw": 32, "ticks": 8},
        # grouped convolutions, 34 million parameters, K = 4, bf16
        {"name": "resnext29_bf16", "kind": "pipeline", "net": "resnext29", "dtype": "bf16", "batch": 128, "hw": 32, "ticks": 32},
        # the headline workload: ImageNet-shaped ResNet-18, K = 4, batch 256, bf16
        {"name": "resnet18_bf16", "kind": "pipeline", "net": "resnet18", "dtype": "bf16", "batch": 256, "hw": 224, "ticks": 32},
        # the same network on a batch and a picture size that fill no tile evenly
        {"name": "resnet18_bf16_ragged", "kind": "pipeline", "net": "resnet18", "dtype": "bf16", "batch": 75, "hw": 174,
         "ticks": 32},
        # one bottleneck stage at ImageNet shape, staleness 3, bf16
        {"name": "conv4x_bf16", "kind": "block", "net": "resnet50_conv4x", "dtype": "bf16", "batch": 64, "hw": 28, "ticks": 32,
         "separate": False},
        # the same stage with a ragged batch on an odd map, the three calls of a step made one by one
        {"name": "conv4x_bf16_ragged", "kind": "block", "net": "resnet50_conv4x", "dtype": "bf16", "batch": 19, "hw": 31,
         "ticks": 32, "separate": True},
        # a deep layer of a CIFAR network: many channels on a small map
        {"name": "layer_bf16_512x4x4", "kind": "layer", "dtype": "bf16", "n": 128, "h": 4, "w": 4, "cin": 512, "cout": 512,
         "k": 3, "stride": 1, "groups": 1, "residual": True},
        # odd sizes throughout, fp32
        {"name": "layer_fp32_odd", "kind": "layer", "dtype": "fp32", "n": 37, "h": 23, "w": 17, "cin": 40, "cout": 72, "k": 3,
         "stride": 2, "groups": 1, "residual": False},
        # the widest pointwise layer of a bottleneck stage
        {"name": "layer_bf16_1x1", "kind": "layer", "dtype": "bf16", "n": 61, "h": 14, "w": 14, "cin": 1024, "cout": 256, "k": 1,
         "stride": 1, "groups": 1, "residual": False},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pipeline", "pipeline", "block", "layer", "layer"])
    if kind == "pipeline":
        net, dtype = rng.choice([("tiny2", "fp32"), ("resnet20", "fp32"), ("resnet56", "bf16"), ("resnet56", "fp32"),
                                 ("vgg19", "bf16"), ("resnext29", "bf16"), ("resnet18", "bf16"), ("resnet18", "bf16")])
        if net == "resnet18":
            batch, hw, ticks = _log(rng, 16, 224), rng.randint(96, 224), 32
        elif net == "resnext29":
            batch, hw, ticks = _log(rng, 16, 128), rng.randint(20, 32), 16
        elif net == "vgg19":
            batch, hw, ticks = _log(rng, 16, 256), rng.choice([32, 32, 48]), 32
        else:
            batch, hw, ticks = _log(rng, 16 if dtype == "bf16" else 8, 256), rng.randint(16, 40), 16
        return {"kind": kind, "net": net, "dtype": dtype, "batch": batch, "hw": hw, "ticks": ticks}
    if kind == "block":
        return {"kind": kind, "net": "resnet50_conv4x", "dtype": "bf16", "batch": _log(rng, 8, 96), "hw": rng.randint(20, 40),
                "ticks": 32, "separate": rng.random() < 0.5}
    dtype = rng.choice(["bf16", "bf16", "fp32"])
    k = rng.choice([1, 3, 3])
    while True:
        h, cin, cout = _log(rng, 4, 56), _log(rng, 16, 1024), _log(rng, 16, 1024)
        if rng.random() < 0.75:  # most layers have whole 16-byte runs of channels
            cin, cout = max(16, cin // 16 * 16), max(16, cout // 16 * 16)
        n, w = _log(rng, 8, 256), max(3, h + rng.randint(-2, 2))
        flops = 2.0 * n * h * w * cin * cout * k * k
        if 2e8 <= flops <= 1.5e11 and n * h * w * max(cin, cout) <= 1 << 26:
            break
    groups = 8 if cin % 128 == 0 and cout % 128 == 0 and rng.random() < 0.25 else 1
    return {"kind": kind, "dtype": dtype, "n": n, "h": h, "w": w, "cin": cin, "cout": cout, "k": k,
            "stride": 2 if h >= 8 and rng.random() < 0.25 else 1, "groups": groups,
            "residual": cout % 8 == 0 and rng.random() < 0.5}


# ----------------------------------------------------------------------------- what a program has in hand
def _code(case):
    return D.DSP_BF16 if case["dtype"] == "bf16" else D.DSP_FP32


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _params(layers, gen):
    """Kaiming-normal weights, gamma = 1, beta = 0, bias 0: per layer a dict of host arrays."""
    out = []
    for shapes in param_shapes(layers):
        d = {}
        for name, shp in shapes:
            if name == "w":
                std = math.sqrt(2.0 / float(np.prod(shp[1:])))
                d[name] = (torch.randn(shp, generator=gen, device="cuda") * std).cpu().numpy()
            else:
                d[name] = (np.ones if name == "gamma" else np.zeros)(shp, np.float32)
        out.append(d)
    return out


def _map(shape, gen, dtype, std=1.0):
    """A feature map of NCHW ``shape`` with values ~ N(0, std^2), as the library takes it (NHWC)."""
    n, c, h, w = shape
    return (torch.randn((n, h, w, c), generator=gen, device="cuda") * std).to(dtype)


class _Training:
    """The library objects of one training run; gives its device memory back when it goes."""

    def __init__(self, case, seed):
        self.case, self.code = case, _code(case)
        self.cfg = cfg = get_config(case["net"], batch=case["batch"], hw=case["hw"])
        gen, td = _generator(seed), _torch_dtype(case)
        self.pl, self.tick = None, 0
        self.blocks = build_gpu_blocks(cfg, [_params(layers, gen) for layers in cfg["blocks"]], self.code)
        shapes = block_shapes(cfg)
        self.batches = [_map(shapes[0], gen, td) for _ in range(_BATCHES)]
        if case["kind"] == "pipeline":
            self.labels = [torch.randint(0, cfg["classes"], (case["batch"],), generator=gen, device="cuda", dtype=torch.int32)
                           for _ in range(_BATCHES)]
            self.pl = D.dsp_pipeline_init(self.blocks, cfg["p"], cfg["m"], _LR, cfg["beta"], cfg["wd"], _MAX_TICKS)
            fill = max(sum(cfg["p"][:k]) + cfg["m"][k] for k in range(cfg["K"]))
        else:
            self.gout = [_map(shapes[1], gen, td, _GRAD_STD) for _ in range(_BATCHES)]
            self.out, self.gin = torch.empty_like(self.gout[0]), torch.empty_like(self.batches[0])
            fill = cfg["m"][0]
        for _ in range(fill + 2):  # fills the queues and takes the first full steps
            self.step(False)

    def step(self, want_loss):
        i = self.tick % _BATCHES
        self.tick += 1
        if self.pl is not None:
            return D.dsp_pipeline_step(self.pl, self.batches[i], self.labels[i], want_loss)[0]
        b, cfg, a, back = self.blocks[0], self.cfg, self.tick - 1, self.tick - 1 - self.cfg["m"][0]
        if back < 0:
            D.dsp_block_forward(b, a, self.batches[i], self.out)
            return None
        if self.case["separate"]:
            D.dsp_block_forward(b, a, self.batches[i], self.out)
            D.dsp_block_recompute_backward(b, back, self.gout[i], self.gin)
        else:
            D.dsp_block_step(b, a, self.batches[i], self.out, None, None, back, self.gout[i], self.gin)
        D.dsp_param_update(b, _LR, cfg["beta"], cfg["wd"])
        return None

    def weights(self):
        return [D.dsp_block_get_params(b) for b in self.blocks]

    def __del__(self):
        if getattr(self, "pl", None) is not None:
            D.dsp_pipeline_destroy(self.pl)
        destroy_blocks(getattr(self, "blocks", []))


def _backward_filters(w, stride, pad, groups):
    """The filter copy backward-data reads, from w[cout][r][s][cin / groups]: wf[cin][R-1-r][S-1-s][cout / groups], for
    stride 2 stored class by class of the parity of the input pixel."""
    co, r, s, ci = w.shape
    wf = w.flip(1, 2).reshape(groups, co // groups, r, s, ci).permute(0, 4, 2, 3, 1).reshape(groups * ci, r, s, co // groups)
    if stride == 1:
        return wf.contiguous()
    parts = [wf[:, (r - 1 - pad - ph) % 2::2, (s - 1 - pad - pw) % 2::2].reshape(-1) for ph in range(2) for pw in range(2)]
    return torch.cat(parts).contiguous()


class _Layer:
    """Tensors, workspaces and sizes of one convolution + batch norm + ReLU."""

    def __init__(self, c, seed):
        gen, td = _generator(seed), _torch_dtype(c)
        self.case, self.code = c, _code(c)
        k, st, g = c["k"], c["stride"], c["groups"]
        pad = k // 2
        self.ho, self.wo = (c["h"] + 2 * pad - k) // st + 1, (c["w"] + 2 * pad - k) // st + 1
        self.m = c["n"] * self.ho * self.wo
        self.conv = (c["n"], c["h"], c["w"], c["cin"], c["cout"], k, k, st, pad, g)
        y = (c["n"], c["cout"], self.ho, self.wo)
        self.x = _map((c["n"], c["cin"], c["h"], c["w"]), gen, td).relu_()  # what the layer below left
        self.dz = _map(y, gen, td, 0.01)
        self.res = _map(y, gen, td) if c["residual"] else None
        w = torch.randn((c["cout"], k, k, c["cin"] // g), generator=gen, device="cuda") * math.sqrt(2.0 * g / (c["cin"] * k * k))
        self.w, self.wt = w.to(td), _backward_filters(w.to(td), st, pad, g)
        self.gamma = torch.ones(c["cout"], device="cuda") + 0.1 * torch.randn(c["cout"], generator=gen, device="cuda")
        self.beta = 0.1 * torch.randn(c["cout"], generator=gen, device="cuda")
        self.bn_x, self.dy = _map(y, gen, td), _map(y, gen, td, 0.01)
        self.y, self.z, self.bn_dx = (torch.empty_like(self.dz) for _ in range(3))
        self.dres = torch.empty_like(self.dz) if c["residual"] else None
        self.dx, self.dw = torch.empty_like(self.x), torch.empty_like(w)
        self.mean, self.invstd, self.dgamma, self.dbeta = (torch.empty_like(self.gamma) for _ in range(4))
        bits = D.dsp_bn_relu_bits_bytes(self.code, self.m, c["cout"]) if c["residual"] else 0
        self.bits = torch.empty(bits, dtype=torch.uint8, device="cuda") if bits else None
        self.wg_bytes = D.dsp_grouped_conv_workspace_bytes(*self.conv)
        self.wg = torch.empty(max(16, self.wg_bytes), dtype=torch.uint8, device="cuda")
        self.bn_bytes = D.dsp_bn_workspace_bytes(c["cout"])
        self.bn = torch.empty(self.bn_bytes, dtype=torch.uint8, device="cuda")

    def step(self):
        code, m, cout = self.code, self.m, self.case["cout"]
        D.dsp_grouped_conv_forward(code, self.x, self.w, self.y, *self.conv)
        if self.bits is not None:
            D.dsp_bn_forward_bits(code, self.bn_x, self.res, self.z, self.gamma, self.beta, 1e-5, m, cout, self.mean, self.invstd,
                                  self.bits, self.bn, self.bn_bytes)
            D.dsp_bn_backward_bits(code, self.dz, self.bn_x, self.bits, self.bn_dx, self.dres, False, False, self.gamma, self.mean,
                                   self.invstd, self.dgamma, self.dbeta, m, cout, self.bn, self.bn_bytes)
        else:
            D.dsp_bn_forward(code, self.bn_x, self.res, self.z, self.gamma, self.beta, 1e-5, m, cout, True, self.mean, self.invstd,
                             self.bn, self.bn_bytes)
            D.dsp_bn_backward(code, self.dz, self.bn_x, self.z, self.bn_dx, self.dres, False, False, self.gamma, self.mean,
                              self.invstd, self.dgamma, self.dbeta, m, cout, True, self.bn, self.bn_bytes)
        D.dsp_grouped_conv_backward_data(code, self.dy, self.wt, self.dx, *self.conv)
        D.dsp_grouped_conv_backward_weight(code, self.x, self.dy, self.dw, *self.conv, self.wg, self.wg_bytes)
        return {"y": self.y, "z": self.z, "bn_dx": self.bn_dx, "dres": self.dres, "dx": self.dx, "dw": self.dw,
                "dgamma": self.dgamma, "dbeta": self.dbeta}


def prepare(case, seed):
    return _Layer(case, seed) if case["kind"] == "layer" else _Training(case, seed)


# ----------------------------------------------------------------------------- one pass
def run(state):
    case = state.case
    if case["kind"] == "layer":
        return state.step()
    loss = None
    for t in range(case["ticks"]):
        loss = state.step(want_loss=t == case["ticks"] - 1)
    if case["kind"] == "pipeline":
        return {"loss": loss, "weights": state.weights()}
    # the gradient handed down is formed too, but after eighteen rectifiers decided on bf16 maps it differs by 30 % between two
    # roundings of the same weights: what makes it up is compared in the layer cases and through the weights
    return {"out": state.out, "weights": state.weights()}


# ----------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "layer":
        k, st, g = case["k"], case["stride"], case["groups"]
        ho, wo = (case["h"] + 2 * (k // 2) - k) // st + 1, (case["w"] + 2 * (k // 2) - k) // st + 1
        x, y = case["n"] * case["h"] * case["w"] * case["cin"], case["n"] * ho * wo * case["cout"]
        w = case["cout"] * k * k * case["cin"] // g
        # in: x, dy, both filter copies, the batch norm's x and dz (and its residual); out: y, dx, dw, the batch norm's z and dx
        # (and its residual's gradient)
        return {"bytes": e * (2 * x + 6 * y + 2 * w + (2 * y if case["residual"] else 0)) + 4 * w,
                "flops": 3 * 2.0 * case["n"] * ho * wo * case["cout"] * k * k * (case["cin"] // g)}
    cfg = get_config(case["net"], batch=case["batch"], hw=case["hw"])
    shapes = block_shapes(cfg)
    flops = traffic = saved = 0.0
    for k, layers in enumerate(cfg["blocks"]):
        n_params = sum(int(np.prod(shp)) for ps in param_shapes(layers) for _, shp in ps)
        for L, s in zip(layers, infer_shapes(layers, shapes[k])):
            if L["op"] == "conv":
                macs = float(np.prod(s)) * L["cin"] // L.get("groups", 1) * L["r"] * L["s"]
            elif L["op"] == "linear":
                macs = float(np.prod(s)) * L["cin"]
            else:
                continue
            data_layer = L["in"] == -1 and k == 0 and cfg.get("data_input", True)
            # forward, recompute of the stale mini-batch, gradient of the weights, gradient of the input
            flops += 2 * macs * (1 + (cfg["m"][k] > 0) + 1 + (not data_layer))
        # the input of a block is written once and read by its forward and by its recompute, the gradient written and read
        # once; weights and momentum are read and written once
        traffic += e * float(np.prod(shapes[k])) * (3 + 2 * (k > 0 or case["kind"] == "block")) + 16.0 * n_params
        saved += 4.0 * n_params
    if case["kind"] == "block":
        traffic += 2 * e * float(np.prod(shapes[-1]))
    return {"bytes": traffic * case["ticks"] + saved, "flops": flops * case["ticks"]}


# How far two runs come apart whose initial parameters differ by one part in 1e7 (that is: whose sums are rounded in another
# order), measured over the ranges above, times about four.  Rounding moves a rectifier here and there, which moves the next
# step's gradient, so the figure belongs to the depth of a network and falls with the batch it averages over; it is given at
# batch 128.  One pass moves the weights by several times as much.
_DRIFT = {("tiny2", "fp32"): 2e-6, ("resnet20", "fp32"): 1e-5, ("resnet56", "fp32"): 3e-4, ("resnet56", "bf16"): 5e-3,
          ("resnet164", "fp32"): 4e-3, ("vgg19", "bf16"): 3e-2, ("resnext29", "bf16"): 4e-3, ("resnet18", "bf16"): 5e-4}


def tolerance(case):
    if case["kind"] == "layer":
        # one rounding to bf16 is 1.7e-3; fp32 sums against 64-bit ones differ by 2.5e-7, up to 2e-6 of the largest
        return {"rel": 7e-3} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 2e-5}
    if case["kind"] == "block":  # eighteen stored bf16 maps in a row: 2.1e-2 between two roundings of the same weights
        return {"rel": 3e-2, "max": 0.6}
    return {"rel": min(3e-2, _DRIFT[case["net"], case["dtype"]] * 128.0 / case["batch"])}
