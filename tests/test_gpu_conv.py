"""Element-wise parity of the three convolution kernels with the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_1909_02625_amd as D
from oracle import dsp_oracle as O
from tests.gpu_harness import dgrad_filter_copy, from_dev, rel_err, round_like, to_dev

pytestmark = pytest.mark.gpu

# (N, H, W, Cin, Cout, R, S, stride, pad): several tiles, ragged tails, every tile family
SHAPES = [
    (3, 9, 9, 16, 16, 3, 3, 1, 1),      # small-channel tile, M = 243 (ragged)
    (2, 8, 8, 3, 16, 3, 3, 1, 1),       # first conv: Cin = 3 -> element-wise gather path
    (2, 12, 12, 16, 32, 3, 3, 2, 1),    # stride 2, 32-channel tile
    (2, 12, 12, 16, 32, 1, 1, 2, 0),    # projection shortcut
    (5, 7, 7, 64, 64, 3, 3, 1, 1),      # 64-wide tile
    (4, 14, 14, 32, 128, 1, 1, 1, 0),   # 1x1
    (2, 10, 10, 128, 256, 3, 3, 1, 1),  # wide
    (2, 20, 20, 3, 64, 7, 7, 2, 3),     # stem 7x7/2
    (2, 20, 20, 8, 64, 7, 7, 2, 3),     # the same with padded channels: 49 taps on the vector path (two mask words)
    (2, 6, 6, 8, 8, 3, 3, 1, 1),        # channel count below the tile width
    (1, 5, 5, 24, 40, 3, 3, 1, 1),      # channel counts that are no power of two
    (4, 13, 13, 16, 16, 3, 3, 2, 1),    # 16 -> 16 channels, stride 2, several slices with a ragged tail
    (2, 11, 11, 16, 16, 1, 1, 1, 0),    # 16 -> 16 channels, 1x1
    (3, 10, 10, 32, 32, 3, 3, 1, 1),    # 32 -> 32 channels: register-resident filters, two channel groups
    (2, 9, 9, 32, 16, 3, 3, 1, 1),      # 32 -> 16
    (33, 32, 32, 16, 16, 3, 3, 1, 1),   # enough pixel groups that each wave walks several of them
    (3, 11, 9, 16, 24, 3, 3, 2, 1),     # stride 2 on odd map sides: the four parity classes have different sizes
    (2, 12, 12, 32, 64, 1, 1, 2, 0),    # 1x1 stride 2: three of the four classes receive no gradient at all
    (2, 9, 9, 8, 16, 2, 2, 2, 0),       # 2x2 stride 2 without padding: one tap per class
    (2, 14, 14, 8, 8, 5, 5, 2, 2),      # 5x5 stride 2: classes of 3x3, 3x2, 2x3 and 2x2 taps
    # 64 -> 64 channels, 3x3: in bf16 the filters-in-registers kernel (persistent workgroups walking 256-pixel tiles,
    # input rows staged once in LDS); every element compared, M = 65856 with a ragged last tile of 64 pixels
    (21, 56, 56, 64, 64, 3, 3, 1, 1),
    (30, 52, 51, 64, 64, 3, 3, 1, 1),   # the shortest rows that kernel takes (a tile touches 8 input rows), H != W, odd W, M = 79560
    (20, 60, 62, 64, 64, 3, 3, 1, 1),   # the longest (patch rows of 64 pixels are full)
    (65, 32, 32, 64, 64, 3, 3, 1, 1),   # rows too short for it: in bf16 the direct-to-LDS 128x64 tile at a large M
]


def _tol(dtype):
    return 2e-2 if dtype == D.DSP_BF16 else 1e-4


@pytest.mark.parametrize("dtype", [D.DSP_FP32, D.DSP_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv_forward_dgrad_wgrad(shape, dtype):
    N, H, W, Ci, Co, R, S, st, pd = shape
    rng = np.random.default_rng(hash(shape) % 2**32)
    x = round_like(rng.standard_normal((N, Ci, H, W)), dtype)
    w = round_like(rng.standard_normal((Co, Ci, R, S)) * np.sqrt(2.0 / (Ci * R * S)), dtype)
    y_ref = O.conv2d_forward(x, w, st, pd)
    dy = round_like(rng.standard_normal(y_ref.shape), dtype)
    dx_ref = O.conv2d_backward_data(dy, w, x.shape, st, pd)
    dw_ref = O.conv2d_backward_weight(x, dy, w.shape, st, pd)

    td = torch.bfloat16 if dtype == D.DSP_BF16 else torch.float32
    d_x, d_dy = to_dev(x, dtype), to_dev(dy, dtype)
    d_w = torch.from_numpy(w.transpose(0, 2, 3, 1).copy()).to("cuda", td)                      # [co][r][s][ci]
    d_wt = torch.from_numpy(dgrad_filter_copy(w, st, pd)).to("cuda", td)   # [ci][R-1-r][S-1-s][co] (stride 2: by parity class)
    d_y = torch.full((N * y_ref.shape[2] * y_ref.shape[3] * Co,), float("nan"), device="cuda", dtype=td)
    D.dsp_conv_forward(dtype, d_x, d_w, d_y, N, H, W, Ci, Co, R, S, st, pd)
    torch.cuda.synchronize()
    assert rel_err(from_dev(d_y, y_ref.shape), y_ref) < _tol(dtype)
    assert np.abs(from_dev(d_y, y_ref.shape) - y_ref).max() < _tol(dtype) * 10 * max(1.0, np.abs(y_ref).max())

    d_dx = torch.full((N * H * W * Ci,), float("nan"), device="cuda", dtype=td)
    D.dsp_conv_backward_data(dtype, d_dy, d_wt, d_dx, N, H, W, Ci, Co, R, S, st, pd, accumulate=False)
    torch.cuda.synchronize()
    got = from_dev(d_dx, x.shape)
    assert rel_err(got, dx_ref) < _tol(dtype)
    # accumulate: dx += ...
    D.dsp_conv_backward_data(dtype, d_dy, d_wt, d_dx, N, H, W, Ci, Co, R, S, st, pd, accumulate=True)
    torch.cuda.synchronize()
    assert rel_err(from_dev(d_dx, x.shape), 2 * dx_ref) < _tol(dtype)

    ws_bytes = D.dsp_conv_workspace_bytes(N, H, W, Ci, Co, R, S, st, pd)
    ws = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda")
    d_dw = torch.full((Co * R * S * Ci,), float("nan"), device="cuda", dtype=torch.float32)
    D.dsp_conv_backward_weight(dtype, d_x, d_dy, d_dw, N, H, W, Ci, Co, R, S, st, pd, ws, ws_bytes)
    torch.cuda.synchronize()
    dw = d_dw.cpu().numpy().astype(np.float64).reshape(Co, R, S, Ci).transpose(0, 3, 1, 2)
    assert rel_err(dw, dw_ref) < _tol(dtype)
    # run-to-run identical (fixed-order split reduction)
    d_dw2 = torch.empty_like(d_dw)
    D.dsp_conv_backward_weight(dtype, d_x, d_dy, d_dw2, N, H, W, Ci, Co, R, S, st, pd, ws, ws_bytes)
    torch.cuda.synchronize()
    assert torch.equal(d_dw, d_dw2)


# The direct-to-LDS tiles where they can go wrong: rows and output channels that fill no tile, fewer k tiles than a tile
# has LDS stages (K = 64), eight groups of waves of which the last have no k tile (18 of them at K = 576), taps cut by every
# border, and channel counts that are no multiple of a k tile (chunks of one k tile in different taps, a ragged k tail), both
# strides.
DIRECT_TO_LDS = [
    (5, 9, 9, 64, 72, 3, 3, 1, 1),
    (1, 5, 5, 64, 32, 1, 1, 1, 0),
    (2, 4, 4, 128, 8, 3, 3, 1, 1),
    (3, 13, 11, 192, 136, 3, 3, 2, 1),
    (9, 17, 15, 256, 200, 1, 1, 1, 0),
    (16, 24, 24, 64, 128, 3, 3, 1, 1),
    (40, 16, 16, 128, 256, 3, 3, 1, 1),
    (2, 9, 9, 72, 40, 3, 3, 1, 1),
    (3, 11, 10, 104, 264, 3, 3, 2, 1),
    (1, 6, 6, 520, 24, 1, 1, 1, 0),
    (12, 20, 20, 88, 96, 3, 3, 1, 1),
    (2, 7, 7, 24, 32, 5, 5, 1, 2),
]


@pytest.mark.parametrize("shape", DIRECT_TO_LDS, ids=lambda s: "x".join(map(str, s)))
def test_direct_to_lds_tiles(shape):
    test_conv_forward_dgrad_wgrad(shape, D.DSP_BF16)


# The bf16 kernel that keeps the filters of 16- and 32-channel 3x3 layers in registers: fewer pixels than one group of 16, a
# ragged last group, all pairs of channel counts, stride 2, no padding, several groups per wave.
SMALL_3X3 = [
    (1, 3, 3, 16, 16, 3, 3, 1, 1),
    (1, 3, 3, 32, 32, 3, 3, 1, 0),
    (2, 7, 9, 16, 32, 3, 3, 1, 1),
    (2, 7, 9, 32, 16, 3, 3, 2, 1),
    (5, 8, 6, 32, 32, 3, 3, 2, 0),
    (41, 21, 23, 32, 32, 3, 3, 1, 1),
    (37, 29, 31, 16, 32, 3, 3, 1, 2),
]


@pytest.mark.parametrize("shape", SMALL_3X3, ids=lambda s: "x".join(map(str, s)))
def test_filters_in_registers_16_and_32_channels(shape):
    D.dsp_profile_start(64)
    try:
        test_conv_forward_dgrad_wgrad(shape, D.DSP_BF16)
    finally:
        launched = {k["name"] for k in D.dsp_profile_stop()}
    assert "conv3x3_direct<bf16,ci%d>" % shape[3] in launched, launched


# ... and the edges of what it takes: (gathered channels, output channels, stride, output rows and columns, accumulating, taken)
SMALL_3X3_EDGES = [
    (32, 32, 2, 128, 32, False, True), (32, 32, 2, 129, 32, False, False),
    (32, 16, 2, 1024, 32, False, True), (32, 16, 2, 1025, 32, False, False),
    (32, 16, 2, 3071, 32, False, False), (32, 16, 2, 3072, 32, False, True),
    (32, 32, 2, 3071, 32, False, False), (32, 32, 2, 3072, 32, False, True),
    (16, 32, 2, 2048, 32, False, True),
    (32, 32, 1, 1024, 1024, False, True), (32, 32, 1, 1025, 1024, False, False),
    (32, 32, 1, 1025, 1024, True, True), (32, 16, 1, 1025, 1024, False, True),
]


@pytest.mark.parametrize("ci, co, stride, rows, cols, accumulate, taken", SMALL_3X3_EDGES)
def test_filters_in_registers_where_the_tiles_take_over(ci, co, stride, rows, cols, accumulate, taken):
    """An accumulating launch is backward-data (of a co -> ci layer), the others are forward; every element against fp64."""
    h, w = stride * rows, stride * cols
    x = torch.randn((1, h, w, ci), device="cuda").bfloat16()
    f = (torch.randn((co, 3, 3, ci), device="cuda") / (3 * ci ** 0.5)).bfloat16()
    y = torch.ones((1, rows, cols, co), device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    D.dsp_profile_start(16)
    try:
        if accumulate:
            D.dsp_conv_backward_data(D.DSP_BF16, x, f, y, 1, rows, cols, co, ci, 3, 3, 1, 1, accumulate=True)
        else:
            D.dsp_conv_forward(D.DSP_BF16, x, f, y, 1, h, w, ci, co, 3, 3, stride, 1)
        torch.cuda.synchronize()
    finally:
        launched = {k["name"] for k in D.dsp_profile_stop()}
    assert ("conv3x3_direct<bf16,ci%d>" % ci in launched) == taken, launched
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    ref = torch.full((rows * cols, co), float(accumulate), device="cuda", dtype=torch.float64)
    mag = ref.clone()
    for r in range(3):
        for s in range(3):
            a = xp[:, r:r + stride * (rows - 1) + 1:stride, s:s + stride * (cols - 1) + 1:stride].reshape(-1, ci)
            b = f[:, r, s].double().t().contiguous()
            ref += a @ b
            mag += a.abs() @ b.abs()
    # rounding to bf16, and 9 ci + 1 additions in fp32
    assert ((y.double().view(-1, co) - ref).abs() <= 2.0**-8 * ref.abs() + (9 * ci + 2) * 2.0**-24 * mag).all()


@pytest.mark.parametrize("dtype", [D.DSP_FP32, D.DSP_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("co", [16, 32])
def test_backward_data_whose_parity_class_is_a_small_3x3(co, dtype):
    """5x5 / stride 2: the class of even pixels is a 3x3 convolution of co -> 16 channels, the shape of the kernels that keep the
    filters of such layers in registers, but its output rows lie two pixels apart."""
    test_conv_forward_dgrad_wgrad((3, 13, 14, 16, co, 5, 5, 2, 2), dtype)


# Stride-2 backward-data as one launch over the parity classes: (shape, launches).  Maps of one row or column (two classes exist), a 7x7
# filter (classes of up to 16 taps), filters larger than the input, several ragged tiles per class, classes that no tap reaches,
# eight wave groups of which the last have no k tile; one class (a 1x1 map), and channels that are no whole 16-byte runs.
PARITY_CLASSES = [
    ((5, 1, 9, 16, 24, 3, 3, 2, 1), 1), ((3, 9, 1, 24, 16, 3, 3, 2, 1), 1), ((2, 15, 13, 8, 16, 7, 7, 2, 3), 1),
    ((1, 3, 3, 264, 320, 3, 3, 2, 1), 1), ((40, 23, 21, 64, 136, 3, 3, 2, 1), 1), ((6, 33, 31, 264, 72, 1, 1, 2, 0), 1),
    ((2, 7, 5, 40, 64, 3, 3, 2, 1), 1), ((3, 1, 1, 16, 16, 3, 3, 2, 1), 1), ((3, 8, 7, 12, 18, 3, 3, 2, 1), 4),
]


@pytest.mark.parametrize("dtype", [D.DSP_FP32, D.DSP_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape, launches", PARITY_CLASSES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_parity_classes_in_one_launch(shape, launches, dtype):
    test_conv_forward_dgrad_wgrad(shape, dtype)
    N, H, W, Ci, Co, R, S, st, pd = shape
    td = torch.bfloat16 if dtype == D.DSP_BF16 else torch.float32
    ho, wo = (H + 2 * pd - R) // st + 1, (W + 2 * pd - S) // st + 1
    dy, wt = torch.randn(N * ho * wo * Co + 1, device="cuda").to(td), torch.randn(Ci * R * S * Co, device="cuda").to(td)
    dx, dx1 = (torch.full((N * H * W * Ci,), float("nan"), device="cuda", dtype=td) for _ in range(2))
    D.dsp_profile_start(16)
    try:
        D.dsp_conv_backward_data(dtype, dy[:-1], wt, dx, *shape)
        torch.cuda.synchronize()
    finally:
        got = sum(k["launches"] for k in D.dsp_profile_stop())
    assert got == launches
    dy[1:] = dy[:-1].clone()  # the same on tensors that are not 16-byte aligned: class by class, element-wise gathers
    D.dsp_conv_backward_data(dtype, dy[1:], wt, dx1, *shape)
    torch.cuda.synchronize()
    assert rel_err(dx1.double().cpu().numpy(), dx.double().cpu().numpy()) < _tol(dtype)


def test_several_output_tiles_per_workgroup():
    """389 tiles of 256 x 128 for 256 compute units, the last row tile and the channels ragged."""
    D.dsp_profile_start(64)
    try:
        test_conv_forward_dgrad_wgrad((127, 28, 28, 128, 104, 3, 3, 1, 1), D.DSP_BF16)
    finally:
        launched = {k["name"] for k in D.dsp_profile_stop()}
    assert "conv_dma_stream<bf16,BM256,BN128,BK64,8 waves>" in launched, launched


# The stream over output tiles where a workgroup walks several: (shape of the layer, groups, backward-data).  389 tiles and a ragged
# column count; three column tiles, the last of 8 channels; the four parity classes of a stride-2 layer on an odd map, 555-647
# tiles each, whose output rows lie two pixels apart; filters larger than the input (column tiles walked first); groups.
STREAMED = [
    ((127, 28, 28, 104, 128, 3, 3, 1, 1), 1, True),
    ((68, 23, 21, 264, 128, 3, 3, 1, 1), 1, True),
    ((910, 27, 25, 72, 512, 3, 3, 2, 1), 1, True),
    ((13, 16, 16, 1024, 4992, 1, 1, 1, 0), 1, False),
    ((161, 16, 16, 256, 288, 3, 3, 1, 1), 4, False),
]


@pytest.mark.parametrize("shape, groups, kind", [(s, g, k) for s, g, b in STREAMED for k in (("plain", "accumulating") if b else ("forward",))],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_streamed_tiles(shape, groups, kind):
    """Every element against fp64: the rounding to bf16 and an addition in fp32 per product."""
    backward, accumulate = kind != "forward", kind == "accumulating"
    N, H, W, Ci, Co, R, S, st, pd = shape
    ho, wo = (H + 2 * pd - R) // st + 1, (W + 2 * pd - S) // st + 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(R * Ci + Co)
    cg, og = Ci // groups, Co // groups
    a = torch.randn((N, ho, wo, Co) if backward else (N, H, W, Ci), generator=gen, device="cuda").bfloat16()
    w = (torch.randn((Co, R, S, cg), generator=gen, device="cuda") / (R * S * (og if backward else cg)) ** 0.5).bfloat16()
    out = torch.randn((N, H, W, Ci) if backward else (N, ho, wo, Co), generator=gen, device="cuda").bfloat16()
    old = out.double() if accumulate else torch.zeros_like(out, dtype=torch.float64)
    d_w = torch.from_numpy(dgrad_filter_copy(w.float().cpu().numpy().transpose(0, 3, 1, 2), st, pd, groups)).to("cuda", torch.bfloat16) if backward else w
    torch.cuda.synchronize()
    D.dsp_profile_start(16)
    try:
        if backward:
            D.dsp_grouped_conv_backward_data(D.DSP_BF16, a, d_w, out, *shape, groups, accumulate=accumulate)
        else:
            D.dsp_grouped_conv_forward(D.DSP_BF16, a, d_w, out, *shape, groups)
        torch.cuda.synchronize()
    finally:
        launched = {k["name"]: k["launches"] for k in D.dsp_profile_stop()}
    assert launched == {"conv_dma_stream<bf16,BM256,BN128,BK64,8 waves>": st * st}, launched
    # the reference: one product per tap (and group), added up at the pixels of x it reads
    pad = torch.nn.functional.pad
    ref, mag = old.clone(), old.abs()
    if backward:
        ref, mag = pad(ref, (0, 0, pd, pd, pd, pd)), pad(mag, (0, 0, pd, pd, pd, pd))
    src = a.double() if backward else pad(a.double(), (0, 0, pd, pd, pd, pd))
    wd = w.double()
    for r in range(R):
        for s in range(S):
            rows, cols = slice(r, r + st * (ho - 1) + 1, st), slice(s, s + st * (wo - 1) + 1, st)
            for i in range(groups):
                f = wd[i * og:(i + 1) * og, r, s]
                if backward:
                    t = src.reshape(-1, Co)
                    ref[:, rows, cols] += (t @ f).view(N, ho, wo, Ci)
                    mag[:, rows, cols] += (t.abs() @ f.abs()).view(N, ho, wo, Ci)
                else:
                    t, o = src[:, rows, cols, i * cg:(i + 1) * cg].reshape(-1, cg), slice(i * og, (i + 1) * og)
                    f = f.t().contiguous()
                    ref[..., o] += (t @ f).view(N, ho, wo, og)
                    mag[..., o] += (t.abs() @ f.abs()).view(N, ho, wo, og)
    if backward:
        ref, mag = ref[:, pd:pd + H, pd:pd + W], mag[:, pd:pd + H, pd:pd + W]
    k = R * S * (og if backward else cg)
    assert ((out.double() - ref).abs() <= 2.0**-8 * ref.abs() + (k + 2) * 2.0**-24 * mag).all()


# The direct-to-LDS backward-weight tiles where they can go wrong: channels and columns that fill no tile (8 of 64, 136 of
# 128 + 128), fewer rows than one LDS stage and than the stages in flight, a step of 64 pixels that passes several images
# (3 x 3 maps), one that stays inside a row (a row of 70), rows dropped by the stride at an odd edge, and eight slices of the
# 128x128 tile.
BACKWARD_WEIGHT = [
    (1, 3, 3, 8, 8, 3, 3, 1, 1),
    (50, 3, 3, 136, 136, 3, 3, 1, 1),
    (2, 3, 70, 24, 40, 3, 3, 1, 1),
    (3, 5, 71, 40, 264, 3, 3, 2, 1),
    (7, 9, 10, 64, 144, 5, 5, 2, 2),
    (130, 14, 14, 136, 264, 3, 3, 1, 1),
    (33, 12, 12, 520, 256, 1, 1, 1, 0),
    (20, 13, 13, 256, 520, 1, 1, 2, 0),
]


@pytest.mark.parametrize("shape", BACKWARD_WEIGHT, ids=lambda s: "x".join(map(str, s)))
def test_direct_to_lds_backward_weight(shape):
    test_conv_forward_dgrad_wgrad(shape, D.DSP_BF16)


# One layer for every direct-to-LDS tile, forward ("conv_dma_gemm", "conv_dma_stream") and backward-weight ("conv_wgrad_dma"): the tile's name as
# the library reports it, and a shape that fills it neither in rows nor in output channels (nor, in the backward-weight ones,
# in columns).  The tiles are chosen by a model of their durations, so a change of that model may ask for other shapes here.
EVERY_TILE = [
    ("conv_dma_gemm<bf16,BM256,BN256,BK32,8x1 waves>", (90, 35, 14, 64, 144, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM256,BN128,BK64,8x1 waves>", (36, 37, 25, 256, 72, 1, 1, 1, 0)),       # one round, four k tiles
    ("conv_dma_stream<bf16,BM256,BN128,BK64,8 waves>", (36, 37, 25, 640, 72, 1, 1, 1, 0)),       # one round, ten
    ("conv_dma_stream<bf16,BM256,BN128,BK64,8 waves>", (180, 30, 31, 448, 72, 1, 1, 1, 0)),      # three rounds, seven
    ("conv_dma_gemm<bf16,BM256,BN128,BK32,4x1 waves>", (108, 25, 37, 64, 80, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM128,BN128,BK32,8x1 waves>", (18, 34, 27, 64, 72, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM128,BN128,BK64,8x1 waves>", (27, 37, 17, 512, 72, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM128,BN64,BK64,4x1 waves>", (79, 30, 14, 384, 8, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM128,BN64,BK32,4x1 waves>", (107, 13, 12, 64, 8, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM256,BN64,BK32,4x1 waves>", (109, 23, 40, 64, 8, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM64,BN64,BK64,4x1 waves>", (1, 6, 33, 64, 8, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM64,BN64,BK64,4x2 waves>", (87, 3, 34, 1024, 8, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM32,BN32,BK32,1x8 waves>", (3, 8, 7, 64, 8, 3, 3, 1, 1)),
    ("conv_dma_gemm<bf16,BM256,BN256,BK32,8x1 waves,any Ci>", (55, 30, 20, 528, 136, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM256,BN128,BK32,4x1 waves,any Ci>", (117, 24, 39, 528, 40, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM128,BN128,BK32,8x1 waves,any Ci>", (37, 12, 37, 520, 88, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM64,BN64,BK32,4x1 waves,any Ci>", (79, 11, 20, 560, 40, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM64,BN64,BK32,4x2 waves,any Ci>", (22, 12, 35, 24, 40, 5, 5, 1, 2)),
    ("conv_dma_gemm<bf16,BM32,BN32,BK32,1x8 waves,any Ci>", (3, 3, 3, 200, 8, 3, 3, 1, 1)),
    ("conv_dma_gemm<bf16,BM128,BN32,BK32,2x2 waves,any Ci>", (117, 19, 16, 568, 8, 1, 1, 1, 0)),
    ("conv_dma_gemm<bf16,BM64,BN32,BK32,2x2 waves,any Ci>", (63, 6, 23, 600, 8, 1, 1, 1, 0)),
    ("conv_wgrad_dma<bf16,BM256,BN128,BK64>", (1, 3, 3, 832, 864, 3, 3, 1, 1)),
    ("conv_wgrad_dma<bf16,BM256,BN128,BK64>", (19, 11, 19, 408, 272, 3, 3, 1, 1)),  # four slices, two chains each
    ("conv_wgrad_dma<bf16,BM128,BN128,BK64>", (1, 3, 4, 576, 192, 5, 5, 1, 2)),
    ("conv_wgrad_dma<bf16,BM64,BN64,BK64>", (2, 12, 25, 8, 8, 1, 1, 1, 0)),
]


@pytest.mark.parametrize("tile, shape", EVERY_TILE, ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_every_direct_to_lds_tile(tile, shape):
    D.dsp_profile_start(64)
    try:
        test_conv_forward_dgrad_wgrad(shape, D.DSP_BF16)
    finally:
        launched = {k["name"] for k in D.dsp_profile_stop()}
    assert tile in launched, launched


# (shape, the longest run of pixels added up as one fp32 chain, slices): the slices of the register-staged rule, whatever
# number of workgroups the direct-to-LDS tiles are dealt out to.
CHAINS = [
    ((128, 4, 4, 512, 512, 3, 3, 1, 1), 704, 3),
    ((21, 12, 13, 144, 688, 3, 3, 1, 1), 512, 7),
]


@pytest.mark.parametrize("offset", [0, 4], ids=["aligned", "unaligned"])
@pytest.mark.parametrize("shape, rows, slices", CHAINS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_backward_weight_rounds_as_short_chains(shape, rows, slices, offset):
    """Rounding a sum to fp32 is off by 0.425 * 2^-24 of it (rms over the mantissas).  The partial sums of a chain of n matrix
    instructions (16 independent products each) grow as sqrt(j / n), so the chain is off by 0.425 * 2^-24 * sqrt((n + 1) / 2) of
    its result, and adding up s of them by sqrt((s + 1) / 2) of that unit more; 15 % on top for the roundings inside an
    instruction.  One chain over all pixels is beyond it."""
    N, H, W, Ci, Co, R, S, st, pd = shape
    rng = np.random.default_rng(23)
    x = round_like(rng.standard_normal((N, Ci, H, W)), D.DSP_BF16)
    dy = round_like(rng.standard_normal((N, Co, H, W)), D.DSP_BF16)
    xp = np.pad(x.transpose(0, 2, 3, 1).astype(np.float64), ((0, 0), (pd, pd), (pd, pd), (0, 0)))
    dym = dy.transpose(0, 2, 3, 1).reshape(-1, Co).astype(np.float64)
    ref = np.stack([dym.T @ xp[:, r:r + H, s:s + W].reshape(-1, Ci) for r in range(R) for s in range(S)], axis=1)
    buf = torch.zeros(N * H * W * Ci + 8, device="cuda", dtype=torch.bfloat16)
    d_x = buf[offset:offset + N * H * W * Ci]
    d_x.copy_(to_dev(x, D.DSP_BF16).view(-1))
    ws_bytes = D.dsp_conv_workspace_bytes(*shape)
    ws = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda")
    d_dw = torch.full((Co * R * S * Ci,), float("nan"), device="cuda", dtype=torch.float32)
    D.dsp_conv_backward_weight(D.DSP_BF16, d_x, to_dev(dy, D.DSP_BF16), d_dw, *shape, ws, ws_bytes)
    torch.cuda.synchronize()
    bound = 1.15 * 0.425 * 2.0 ** -24 * np.sqrt((rows / 16 + 1) / 2 + (slices + 1) / 2)
    err = rel_err(d_dw.cpu().numpy().reshape(ref.shape), ref)
    assert err < bound


# Filters as wide as a row's mask of taps has bits: 32 taps in one word (direct-to-LDS tiles), 64 in two (register-staged).
WHOLE_MASK_ROWS = [
    (2, 3, 40, 64, 64, 1, 32, 1, 0),
    (2, 3, 37, 40, 16, 1, 32, 1, 0),
    (1, 2, 70, 8, 16, 1, 64, 1, 0),
]


@pytest.mark.parametrize("dtype", [D.DSP_FP32, D.DSP_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", WHOLE_MASK_ROWS, ids=lambda s: "x".join(map(str, s)))
def test_filter_row_that_fills_the_tap_mask(shape, dtype):
    test_conv_forward_dgrad_wgrad(shape, dtype)


# fp32, 128 x 64 tiles with k steps of 16 and, above a contraction of 64, of 32; ragged rows, channels and contractions.
SHORT_CONTRACTIONS = [((49, 32, 33, 16, 64, 1, 1, 1, 0), 16), ((51, 32, 33, 64, 40, 1, 1, 1, 0), 16), ((50, 33, 32, 4, 60, 3, 3, 1, 1), 16),
                      ((51, 32, 33, 68, 40, 1, 1, 1, 0), 32)]


@pytest.mark.parametrize("shape, bk", SHORT_CONTRACTIONS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_short_contractions_fp32(shape, bk):
    D.dsp_profile_start(64)
    try:
        test_conv_forward_dgrad_wgrad(shape, D.DSP_FP32)
    finally:
        names = {k["name"] for k in D.dsp_profile_stop()}
    assert "conv_gather_gemm<fp32,mfma32,BM128,BN64,BK%d,vec>" % bk in names, names


# bf16 backward-weight with one 16 x 16 block of channels per workgroup: (N, H, W, Cin, Cout, stride), taken.  One pixel; one column; several
# images a tile, the last tile short; tiles of part of an image, the last one short; the widest row and the next; more channels, channels
# that make no block, a stride; the fewest pixels and one less.
NARROW = [
    ((520, 1, 1, 16, 16, 1), True), ((103, 5, 1, 32, 16, 1), True), ((3, 9, 19, 32, 16, 1), True), ((2, 16, 16, 16, 16, 1), False),
    ((29, 7, 9, 16, 32, 1), True), ((5, 43, 31, 16, 16, 1), True),
    ((1, 9, 128, 16, 16, 1), True), ((2, 9, 129, 16, 16, 1), False), ((9, 12, 11, 32, 32, 1), True), ((9, 12, 11, 48, 16, 1), False),
    ((2, 9, 9, 16, 24, 1), False), ((4, 29, 30, 32, 16, 2), False),
]


@pytest.mark.parametrize("shape, taken", NARROW, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_backward_weight_by_channel_blocks(shape, taken):
    dtype, td = D.DSP_BF16, torch.bfloat16
    N, H, W, Ci, Co, st = shape
    ho, wo = (H - 1) // st + 1, (W - 1) // st + 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * W)
    x, dy = torch.randn((N, H, W, Ci), generator=gen, device="cuda").to(td), torch.randn((N, ho, wo, Co), generator=gen, device="cuda").to(td)
    full = (N, H, W, Ci, Co, 3, 3, st, 1)
    ws_bytes = D.dsp_conv_workspace_bytes(*full)
    ws = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda")
    for infinite in (False, True):
        if infinite:  # in the corners of the map: it reaches the taps that read them and no others
            x[0, 0, W - 1, 3] = x[0, H - 1, 0, 5] = float("inf")
        dw = torch.full((Co, 3, 3, Ci), float("nan"), device="cuda")
        D.dsp_profile_start(16)
        try:
            D.dsp_conv_backward_weight(dtype, x, dy, dw, *full, ws, ws_bytes)
            torch.cuda.synchronize()
        finally:
            names = {k["name"] for k in D.dsp_profile_stop()}
        assert ("conv_wgrad_narrow<bf16,16x16>" in names) == taken, names
        xp, d = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1)), dy.double().reshape(-1, Co)
        ref, mag = torch.empty((Co, 3, 3, Ci), device="cuda", dtype=torch.float64), torch.empty((Co, 3, 3, Ci), device="cuda", dtype=torch.float64)
        for r in range(3):
            for s in range(3):
                a = xp[:, r:r + st * (ho - 1) + 1:st, s:s + st * (wo - 1) + 1:st].reshape(-1, Ci)
                finite = torch.where(a.isinf(), torch.zeros_like(a), a)
                ref[:, r, s], mag[:, r, s] = d.t().contiguous() @ finite, d.abs().t().contiguous() @ finite.abs()
                ref[:, r, s][:, a.isinf().any(0)] = float("inf")
        hit = ref.isinf()
        assert torch.equal(~dw.isfinite(), hit)
        if not infinite or H * W > 1:
            # an fp32 addition per pixel (products of bf16 values are exact)
            assert ((dw.double() - ref).abs() <= (N * ho * wo + 1) * 2.0**-24 * mag)[~hit].all()


# (N, H, W, Cin, Cout, R, S, stride, pad, groups)
GROUPED = [
    (3, 9, 9, 32, 48, 3, 3, 1, 1, 4),       # 8 -> 12 channels per group: bf16 rows of the output are no whole 16-byte runs
    (2, 12, 12, 64, 64, 3, 3, 2, 1, 8),     # stride 2 (parity classes per group)
    (2, 8, 8, 128, 128, 3, 3, 1, 1, 2),     # 64 -> 64 per group
    (2, 6, 6, 12, 6, 1, 1, 1, 0, 3),        # 4 -> 2 per group: element-wise paths
    (2, 7, 7, 16, 16, 3, 3, 1, 1, 16),      # depthwise
    (2, 10, 10, 512, 512, 3, 3, 1, 1, 8),   # ResNeXt-29 (8 x 64d) stage 1
    (1, 9, 9, 256, 256, 3, 3, 2, 1, 8),     # 32 -> 32 per group, stride 2, odd sides
    (5, 6, 6, 24, 64, 1, 1, 1, 0, 2),       # 12 -> 32 per group
    # direct-to-LDS tiles whose k tiles straddle taps: 72 -> 40, 72 -> 40, 80 -> 32 and 112 -> 32 per group
    (26, 9, 9, 144, 80, 3, 3, 1, 1, 2),
    (21, 10, 10, 288, 160, 3, 3, 1, 1, 4),
    (1, 4, 4, 160, 64, 3, 3, 1, 1, 2),
    (21, 20, 20, 224, 64, 3, 3, 1, 1, 2),
]


@pytest.mark.parametrize("dtype", [D.DSP_FP32, D.DSP_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", GROUPED, ids=lambda s: "x".join(map(str, s)))
def test_grouped_conv_forward_dgrad_wgrad(shape, dtype):
    """The three kernels on grouped convolutions against the oracle's (one ordinary convolution per group); tensors start
    as NaN so that a channel a group forgot to write shows."""
    N, H, W, Ci, Co, R, S, st, pd, G = shape
    rng = np.random.default_rng(hash(shape) % 2**32)
    x = round_like(rng.standard_normal((N, Ci, H, W)), dtype)
    w = round_like(rng.standard_normal((Co, Ci // G, R, S)) * np.sqrt(2.0 * G / (Ci * R * S)), dtype)
    y_ref = O.conv2d_forward(x, w, st, pd, G)
    dy = round_like(rng.standard_normal(y_ref.shape), dtype)
    dx_ref = O.conv2d_backward_data(dy, w, x.shape, st, pd, G)
    dw_ref = O.conv2d_backward_weight(x, dy, w.shape, st, pd, G)

    td = torch.bfloat16 if dtype == D.DSP_BF16 else torch.float32
    d_x, d_dy = to_dev(x, dtype), to_dev(dy, dtype)
    d_w = torch.from_numpy(w.transpose(0, 2, 3, 1).copy()).to("cuda", td)         # [co][r][s][ci within the group]
    d_wt = torch.from_numpy(dgrad_filter_copy(w, st, pd, G)).to("cuda", td)
    d_y = torch.full((N * y_ref.shape[2] * y_ref.shape[3] * Co,), float("nan"), device="cuda", dtype=td)
    D.dsp_grouped_conv_forward(dtype, d_x, d_w, d_y, N, H, W, Ci, Co, R, S, st, pd, G)
    torch.cuda.synchronize()
    assert rel_err(from_dev(d_y, y_ref.shape), y_ref) < _tol(dtype)

    d_dx = torch.full((N * H * W * Ci,), float("nan"), device="cuda", dtype=td)
    D.dsp_grouped_conv_backward_data(dtype, d_dy, d_wt, d_dx, N, H, W, Ci, Co, R, S, st, pd, G, accumulate=False)
    torch.cuda.synchronize()
    assert rel_err(from_dev(d_dx, x.shape), dx_ref) < _tol(dtype)
    D.dsp_grouped_conv_backward_data(dtype, d_dy, d_wt, d_dx, N, H, W, Ci, Co, R, S, st, pd, G, accumulate=True)
    torch.cuda.synchronize()
    assert rel_err(from_dev(d_dx, x.shape), 2 * dx_ref) < _tol(dtype)

    ws_bytes = D.dsp_grouped_conv_workspace_bytes(N, H, W, Ci, Co, R, S, st, pd, G)
    ws = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda")
    d_dw = torch.full((Co * R * S * (Ci // G),), float("nan"), device="cuda", dtype=torch.float32)
    D.dsp_grouped_conv_backward_weight(dtype, d_x, d_dy, d_dw, N, H, W, Ci, Co, R, S, st, pd, G, ws, ws_bytes)
    torch.cuda.synchronize()
    dw = d_dw.cpu().numpy().astype(np.float64).reshape(Co, R, S, Ci // G).transpose(0, 3, 1, 2)
    assert rel_err(dw, dw_ref) < _tol(dtype)
    with pytest.raises(D.DSPError):
        D.dsp_grouped_conv_forward(dtype, d_x, d_w, d_y, N, H, W, Ci, Co, R, S, st, pd, 5 if G != 5 else 7)  # 5 divides no case


def test_conv_rejects_bad_arguments():
    x = torch.zeros(16, device="cuda")
    with pytest.raises(D.DSPError):
        D.dsp_conv_forward(D.DSP_FP32, x, x, x, 1, 2, 2, 4, 4, 3, 3, 0, 1)  # stride 0
    with pytest.raises(D.DSPError):
        D.dsp_conv_backward_data(D.DSP_FP32, x, x, x, 1, 8, 8, 4, 4, 3, 3, 3, 1)  # stride 3 unsupported
    with pytest.raises(D.DSPError):
        D.dsp_conv_backward_weight(D.DSP_FP32, x, x, x, 64, 32, 32, 16, 16, 3, 3, 1, 1, None, 0)  # no workspace


# ---- the layer shapes of the benchmark configurations at their full sizes ------------------------------
# The large tiles (128x128, 128x64, the 128x128 backward-weight tile, the dilated vector kernel) and
# the launch shapes bench.py times only occur at these sizes, where the full fp64 convolution would take
# minutes: a sample of output elements is checked, each computed by the oracle from the definition, plus
# the corners of every tensor (first / last image, channel and pixel: tile and slice tails).
FULL = [
    (D.DSP_FP32, 128, 32, 32, 16, 16, 3, 3, 1, 1),     # ResNet-20/56 stage 1 (register-resident filters, streaming wgrad)
    (D.DSP_FP32, 128, 16, 16, 32, 32, 3, 3, 1, 1),     # stage 2
    (D.DSP_FP32, 128, 8, 8, 64, 64, 3, 3, 1, 1),       # stage 3
    (D.DSP_FP32, 128, 32, 32, 16, 32, 3, 3, 2, 1),     # stage transition, stride 2 (dilated backward-data)
    (D.DSP_BF16, 64, 14, 14, 256, 256, 3, 3, 1, 1),    # ResNet-50 conv4_x 3x3
    (D.DSP_BF16, 64, 14, 14, 256, 1024, 1, 1, 1, 0),   # its 1x1 expansion
    (D.DSP_BF16, 64, 14, 14, 1024, 256, 1, 1, 1, 0),   # and reduction
    (D.DSP_BF16, 256, 28, 28, 128, 128, 3, 3, 1, 1),   # ResNet-18 stage 2 (direct-to-LDS 256x128 tiles)
    (D.DSP_BF16, 256, 56, 56, 64, 128, 3, 3, 2, 1),    # ResNet-18 stage transition
    (D.DSP_BF16, 256, 7, 7, 512, 512, 3, 3, 1, 1),     # ResNet-18 stage 4 (7x7 maps: pixel runs cross image rows; direct-to-LDS 256x128 tiles)
    (D.DSP_BF16, 256, 14, 14, 256, 256, 3, 3, 1, 1),   # ResNet-18 stage 3 (direct-to-LDS 256x256 tiles)
    (D.DSP_BF16, 250, 14, 14, 256, 256, 3, 3, 1, 1),   # the same with a ragged last row tile (M = 49000)
    (D.DSP_BF16, 125, 14, 14, 256, 384, 3, 3, 1, 1),   # direct-to-LDS 256x256 tiles, the second one half empty, ragged rows
    (D.DSP_BF16, 256, 56, 56, 64, 64, 3, 3, 1, 1),     # ResNet-18 stage 1 (filters in registers, 3136 tiles on 256 workgroups)
    (D.DSP_BF16, 128, 32, 32, 512, 512, 3, 3, 1, 1, 8),   # ResNeXt-29 (8 x 64d) stage 1: 8 groups of 64 -> 64
    (D.DSP_BF16, 128, 32, 32, 1024, 1024, 3, 3, 2, 1, 8), # stage 2 entry: 128 -> 128 per group, stride 2
    (D.DSP_FP32, 64, 8, 8, 2048, 2048, 3, 3, 1, 1, 8),    # stage 3: 256 -> 256 per group
]


def _sample(rng, shape, n):
    corners = [tuple(0 for _ in shape), tuple(d - 1 for d in shape)]
    rand = [tuple(int(rng.integers(0, d)) for d in shape) for _ in range(n)]
    return corners + rand


@pytest.mark.parametrize("cfg", FULL, ids=lambda c: ("bf16_" if c[0] == D.DSP_BF16 else "fp32_") + "x".join(map(str, c[1:])))
def test_conv_full_size_sampled(cfg):
    dtype, N, H, W, Ci, Co, R, S, st, pd = cfg[:10]
    G = cfg[10] if len(cfg) > 10 else 1
    rng = np.random.default_rng(1000 + Ci * 7 + Co * 3 + H)
    Ho, Wo = (H + 2 * pd - R) // st + 1, (W + 2 * pd - S) // st + 1
    x = round_like(rng.standard_normal((N, Ci, H, W), dtype=np.float32), dtype)
    w = round_like((rng.standard_normal((Co, Ci // G, R, S)) * np.sqrt(2.0 * G / (Ci * R * S))).astype(np.float32), dtype)
    dy = round_like(rng.standard_normal((N, Co, Ho, Wo), dtype=np.float32), dtype)
    td = torch.bfloat16 if dtype == D.DSP_BF16 else torch.float32
    d_x, d_dy = to_dev(x, dtype), to_dev(dy, dtype)
    d_w = torch.from_numpy(np.ascontiguousarray(w.transpose(0, 2, 3, 1))).to("cuda", td)
    d_wt = torch.from_numpy(dgrad_filter_copy(w, st, pd, G)).to("cuda", td)
    # relative to the typical magnitude of the tensor: stored bf16 has 8 mantissa bits, fp32 sums ~1e-6
    tol = 1e-2 if dtype == D.DSP_BF16 else 1e-4

    d_y = torch.full((N * Ho * Wo * Co,), float("nan"), device="cuda", dtype=td)
    D.dsp_grouped_conv_forward(dtype, d_x, d_w, d_y, N, H, W, Ci, Co, R, S, st, pd, G)
    torch.cuda.synchronize()
    assert not torch.isnan(d_y.float()).any()
    y = d_y.view(N, Ho, Wo, Co)
    idx = _sample(rng, (N, Co, Ho, Wo), 48)
    ref = O.conv2d_forward_at(x, w, st, pd, idx, G)
    got = np.array([float(y[n, ho, wo, k]) for (n, k, ho, wo) in idx])
    scale = max(np.sqrt(np.mean(ref ** 2)), 1e-6)
    assert np.abs(got - ref).max() < tol * 4 * scale, (np.abs(got - ref).max(), scale)

    d_dx = torch.full((N * H * W * Ci,), float("nan"), device="cuda", dtype=td)
    D.dsp_grouped_conv_backward_data(dtype, d_dy, d_wt, d_dx, N, H, W, Ci, Co, R, S, st, pd, G, accumulate=False)
    torch.cuda.synchronize()
    assert not torch.isnan(d_dx.float()).any()
    dx = d_dx.view(N, H, W, Ci)
    idx = _sample(rng, (N, Ci, H, W), 48)
    ref = O.conv2d_backward_data_at(dy, w, x.shape, st, pd, idx, G)
    got = np.array([float(dx[n, hi, wi, c]) for (n, c, hi, wi) in idx])
    scale = max(np.sqrt(np.mean(ref ** 2)), 1e-6)
    assert np.abs(got - ref).max() < tol * 4 * scale, (np.abs(got - ref).max(), scale)

    ws_bytes = D.dsp_grouped_conv_workspace_bytes(N, H, W, Ci, Co, R, S, st, pd, G)
    ws = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda")
    d_dw = torch.full((Co * R * S * (Ci // G),), float("nan"), device="cuda", dtype=torch.float32)
    D.dsp_grouped_conv_backward_weight(dtype, d_x, d_dy, d_dw, N, H, W, Ci, Co, R, S, st, pd, G, ws, ws_bytes)
    torch.cuda.synchronize()
    assert not torch.isnan(d_dw).any()
    dw = d_dw.view(Co, R, S, Ci // G)
    idx = _sample(rng, (Co, Ci // G, R, S), 24)
    ref = O.conv2d_backward_weight_at(x, dy, st, pd, idx, G)
    got = np.array([float(dw[k, r, s, c]) for (k, c, r, s) in idx])
    scale = max(np.sqrt(np.mean(ref ** 2)), 1e-6)
    # fp32 accumulation over N*Ho*Wo products of unit-variance terms
    assert np.abs(got - ref).max() < 1e-3 * scale, (np.abs(got - ref).max(), scale)
