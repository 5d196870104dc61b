"""Kernel variants at the sizes where their tiling can go wrong: tile edges,
remainders, and the smallest and largest shapes of each dispatch rule."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_08300_amd as cs
import variants
from gpu_util import f64, say
from nets import SharedFlatten

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TDT = {"f32": torch.float32, "bf16": torch.bfloat16}


# N, C, H, W, R, S, stride, pad, dilation, groups.  The LDS gather (large matrices, several taps) has tiles of 64
# output columns and 64 (bf16) or 32 (fp32) channels; small matrices, small tiles, rows that are no whole units and
# very long or wide filters keep the other two.
IM2COL = [
    (200, 64, 9, 65, 3, 3, 1, 1, 1, 1),        # one column past a column tile
    (180, 72, 9, 64, 3, 3, 1, 1, 1, 1),         # channel remainder of 8, one full column tile
    (2400, 200, 7, 7, 3, 3, 2, 1, 1, 2),       # groups with a channel remainder, stride 2
    (2100, 8, 130, 3, 1, 1, 1, 0, 1, 1),       # one tap, narrow rows: 16-byte units
    (13000, 512, 1, 1, 1, 1, 1, 0, 1, 1),       # one pixel
    (110, 96, 13, 150, 5, 3, (1, 2), (2, 1), 1, 1),  # mixed strides, 75 columns
    (2000, 92, 5, 5, 3, 3, 1, 1, 1, 1),        # whole small planes, channel remainder
    (2600, 112, 6, 4, 5, 5, (2, 1), 2, 1, 1),  # 12 pixels a tile
    (150, 16, 20, 21, 7, 7, 1, 3, 1, 1),       # 49 taps: smaller channel chunks
    (3, 8, 40, 40, 17, 17, 1, 8, 1, 1),        # 289 units per pixel: the general vector gather
    (1, 16, 150, 150, 3, 3, 1, 60, 60, 1),     # dilation 60: tiles halved until they fit, or the vector gather
    (2, 64, 9, 9, 3, 3, 1, 1, 1, 1),           # a small matrix
    (3, 3, 17, 18, 7, 7, 2, 3, 1, 1),          # 147 elements per row: the element gather
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", IM2COL, ids=str)
def test_im2col_tiles_are_bit_exact(case, dtype):
    N, C, H, W, R, S, st, pd, dl, G = case
    x = torch.randn(N, C, H, W, generator=torch.Generator().manual_seed(3)).to(TDT[dtype])
    say("im2col tiles", case, dtype)
    col = cs.im2col(x.to(DEV), (R, S), st, pd, dl, G)
    torch.cuda.synchronize()
    assert np.array_equal(f64(col), oracle.im2col(f64(x), R, S, st, pd, dl, G))


# Tile columns of the Winograd input transform: 7, 15 and 31 tiles per workgroup, one more and one less;
# channel blocks of 32 with a remainder.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tiles", [1, 6, 7, 8, 14, 15, 16, 28, 31, 32, 45])
def test_winograd_input_transform_tiles(tiles, dtype):
    for W, C, pad in ((2 * tiles, 33, 1), (2 * tiles + 1, 32, 0)):
        if W + 2 * pad < 3:
            continue
        x = torch.randn(2, C, 5, W, generator=torch.Generator().manual_seed(W)).to(TDT[dtype])
        say("winograd input tiles", tiles, W, C, pad, dtype)
        V = cs.winograd_input_transform(x.to(DEV), padding=pad)
        torch.cuda.synchronize()
        ref = oracle.winograd_input_transform(f64(x), padding=pad).reshape(16, -1, C)
        # three adds of fp32 values, then (bf16) one rounding, relative to the largest entry
        tol = 4 * 2.0 ** -24 if dtype == "f32" else 2.0 ** -8
        assert np.abs(f64(V) - ref).max() <= tol * np.abs(ref).max()


# Large fp32 inputs take 15 or 31 tiles per workgroup: tile rows one short of a block, whole, and one over, and a
# channel remainder; 64 lanes only for rows that fill them.
@pytest.mark.parametrize("n,c,w", [(45, 65, 28), (45, 65, 30), (45, 65, 32), (40, 70, 60), (40, 70, 62), (25, 65, 100)])
def test_winograd_input_transform_wide_blocks(n, c, w):
    x = torch.randn(n, c, 28, w, generator=torch.Generator().manual_seed(w))
    say("winograd input wide blocks", n, c, w)
    V = cs.winograd_input_transform(x.to(DEV), padding=1)
    torch.cuda.synchronize()
    ref = oracle.winograd_input_transform(f64(x), padding=1).reshape(16, -1, c)
    assert np.abs(f64(V) - ref).max() <= 4 * 2.0 ** -24 * np.abs(ref).max()


# K, C, H, W of 1x1 IM2COL + GEMM layers: the products' tiles (64 or more rows and columns, k-tiles of 64 bf16 or
# 32 fp32) with remainders on each axis, batches folded and not (planes of 1024 pixels), and reductions that are
# no whole 16-byte units (the register-staged kernel).
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(64, 64, 8, 8), (65, 8, 7, 9), (63, 72, 9, 7), (130, 40, 32, 32), (8, 36, 33, 31),
                                  (257, 200, 16, 17), (5, 7, 6, 6)], ids=str)
def test_gemm_tiles(case, dtype):
    K, C, H, W = case
    g = torch.Generator().manual_seed(K)
    x = torch.randn(3, C, H, W, generator=g).to(TDT[dtype])
    w = torch.randn(K, C, 1, 1, generator=g).to(TDT[dtype])
    b = torch.randn(K, generator=g).to(TDT[dtype])
    say("gemm tiles", case, dtype)
    y = cs.conv2d(x.to(DEV), w.to(DEV), b.to(DEV), algo="im2col_gemm", relu=True)
    torch.cuda.synchronize()
    ref = oracle.conv2d(f64(x), f64(w), f64(b), 1, 0, 1, 1, True)
    # C + 1 fp32 roundings of sums whose terms' absolute values add up to S; bf16: one more of the result
    S = oracle.conv2d(np.abs(f64(x)), np.abs(f64(w)), np.abs(f64(b)), 1, 0, 1, 1, False)
    tol = (C + 1) * 2.0 ** -24 * S + (0 if dtype == "f32" else 2.0 ** -8 * np.abs(ref))
    assert (np.abs(f64(y) - ref) <= tol + 1e-30).all()


class Chain(torch.nn.Module):
    """Two or three convolutions that run channels-last: R x S with stride, padding and dilation, 1 x 1, and
    (with a residual) 3 x 3 back to the first one's channels."""

    def __init__(self, c, k, r, st, pad, dil, k2, res):
        super().__init__()
        self.a = torch.nn.Conv2d(c, k, r, st, pad, dil)
        self.b = torch.nn.Conv2d(k, k2, 1)
        self.c = torch.nn.Conv2d(k2, k, 3, 1, 1)
        self.res = res

    def forward(self, x):
        y = torch.relu(self.a(x))
        z = self.c(torch.relu(self.b(y)))
        return torch.relu(z + y) if self.res else z


# N, C, H, W, K, R, stride, pad, dilation, K2, residual: filters, strides, dilations and residuals on the smaller
# tiles (variants.py reaches every tile); a small copy and a plane of odd size each make the chain channels-last.
CHAINS = [
    (1, 64, 14, 14, 64, 3, 1, 1, 1, 128, True),
    (3, 72, 15, 16, 40, 3, 2, 1, 1, 64, True),
    (1, 8, 9, 10, 16, 5, 1, 2, 1, 8, False),
    (2, 24, 17, 18, 72, 7, 2, 3, 1, 40, True),
    (1, 64, 20, 20, 64, 3, 1, 2, 2, 64, True),
    (5, 16, 7, 8, 200, 1, 1, 0, 1, 136, True),
    (1, 512, 7, 7, 512, 3, 1, 1, 1, 64, False),
    (4, 128, 16, 16, 256, 3, 1, 1, 1, 64, True),
    (40, 64, 14, 14, 256, 1, 1, 0, 1, 64, True),
    (150, 128, 14, 14, 64, 3, 1, 1, 1, 128, False),
    (64, 64, 27, 27, 128, 1, 2, 0, 1, 256, True),
    (16, 8, 45, 45, 64, 3, 1, 1, 1, 512, False),
    (1, 64, 2, 2, 64, 3, 2, 1, 1, 64, True),       # 3 x 3 on a 1 x 1 plane: taps past the whole buffer
]


@pytest.mark.parametrize("case", CHAINS, ids=str)
def test_channels_last_chain(case):
    N, C, H, W, K, R, st, pad, dil, K2, res = case
    torch.manual_seed(C + K)
    net = Chain(C, K, R, st, pad, dil, K2, res).to(torch.bfloat16).eval()
    x = torch.randn(N, C, H, W).to(torch.bfloat16)
    model = cs.swap_backend(net.to(DEV), "implicit_gemm")
    say("channels-last chain", case)
    y = model(x.to(DEV))
    torch.cuda.synchronize()
    assert model.describe().count("channels_last") >= 2
    again = model(x.to(DEV))
    torch.cuda.synchronize()
    assert torch.equal(y, again)

    def conv(v, m, relu):
        o = oracle.conv2d(v, f64(m.weight), f64(m.bias), m.stride[0], m.padding[0], m.dilation[0], 1, relu)
        return torch.from_numpy(o).to(torch.bfloat16).double().numpy()  # stored values are bf16

    a = conv(f64(x), net.a, True)
    z = conv(conv(a, net.b, True), net.c, False)
    ref = np.maximum(z + a, 0) if res else z
    # three bf16 roundings of fp32 sums on each side, the first two spread over sums of the later layers
    assert np.abs(f64(y) - ref).max() <= 3 * 2.0 ** -8 * np.abs(ref).max()


@pytest.mark.parametrize("pooled", [True, False])
def test_linear_beside_a_channels_last_copy(pooled):
    """A linear layer on a flattened image that convolutions read as a channels-last copy."""
    torch.manual_seed(5)
    net = SharedFlatten(pooled).to(torch.bfloat16).eval()
    x = torch.randn(2, 64, *((14, 14) if pooled else (7, 7))).to(torch.bfloat16)
    say("linear beside a channels-last copy", pooled)
    model = cs.swap_backend(net.to(DEV), "implicit_gemm")
    y = model(x.to(DEV))
    torch.cuda.synchronize()
    assert "copy@" in model.describe()
    ref = net.cpu().double()(x.double()).detach().numpy()
    # five bf16 roundings of fp32 sums
    assert np.abs(f64(y) - ref).max() <= 5 * 2.0 ** -8 * np.abs(ref).max()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c,h,w", [(8, 2, 3), (40, 7, 7), (72, 16, 4), (64, 5, 13), (136, 33, 31)])
def test_global_average_is_the_same_in_both_layouts(c, h, w, dtype):
    """Sums of one order: a channels-last average equals the N x C x H x W one in every bit.  Layers that copy their
    input (one filter tap of 1) put the averaged values in either layout."""
    conv, dw = torch.nn.Conv2d(c, c, 1, bias=False), torch.nn.Conv2d(c, c, 3, 1, 1, groups=c, bias=False)
    with torch.no_grad():
        conv.weight.copy_(torch.eye(c)[:, :, None, None])
        dw.weight.zero_()[:, :, 1, 1] = 1.0
    net = torch.nn.Sequential(conv, dw, torch.nn.AdaptiveAvgPool2d(1)).to(TDT[dtype]).eval().to(DEV)
    x = torch.randn(3, c, h, w, generator=torch.Generator().manual_seed(c)).to(TDT[dtype]).to(DEV)
    last = cs.swap_backend(net, ["implicit_gemm", "direct"])
    planes = cs.swap_backend(net, "direct")
    say("global average in both layouts", c, h, w, dtype)
    y, ref = last(x), planes(x)
    torch.cuda.synchronize()
    assert "channels_last" in last.describe() and "channels_last" not in planes.describe()
    assert torch.equal(y, ref)


class EndsInPool(torch.nn.Module):
    def __init__(self):
        super().__init__()
        self.a, self.b, self.pool = torch.nn.Conv2d(16, 32, 1), torch.nn.Conv2d(32, 16, 1), torch.nn.MaxPool2d(7)

    def forward(self, x):
        return self.pool(self.b(self.a(x)))


def test_channels_last_pooling_into_an_unaligned_output():
    """The output tensor of a model needs its elements' alignment only."""
    torch.manual_seed(6)
    net = EndsInPool().to(torch.bfloat16).eval()
    x = torch.randn(3, 16, 7, 7).to(torch.bfloat16)
    model = cs.swap_backend(net.to(DEV), "implicit_gemm")
    xd = x.to(DEV)
    y = model(xd)
    assert model.describe().count("channels_last") == 2
    room = torch.full((3 * 16 + 2,), 7.0, dtype=torch.bfloat16, device=DEV)
    say("channels-last pooling into an unaligned output")
    model._native.forward(xd.data_ptr(), room[1:].data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(room[1:-1].reshape(y.shape), y) and room[0] == 7 and room[-1] == 7


@pytest.mark.parametrize("case", variants.CASES, ids=str)
def test_channels_last_variants(case):
    dtype, n, c, h, w = case[:5]
    torch.manual_seed(c + 3 * case[5])
    net = variants.Pair(*case).eval()
    x = torch.randn(n, c, h, w).to(TDT[dtype])
    say("channels-last variant", case)
    model = variants.lower(case, net.to(DEV))
    y = model(x.to(DEV))
    torch.cuda.synchronize()
    assert model.describe().count("channels_last") >= 2
    net = net.cpu()

    def conv(v, m, relu):
        v = torch.nn.functional.conv2d(v, m.weight.double(), m.bias.double(), m.stride, m.padding, m.dilation,
                                       m.groups)
        return (v.relu() if relu else v).to(TDT[dtype]).double()  # values are stored in the data type

    with torch.no_grad():
        ref = conv(x.double(), net.a, True)
        if dtype == "f32":
            ref = conv(ref, net.dw, True)
        ref = conv(ref, net.b, False)
        if net.res:
            ref = torch.relu(ref + x.double())
    # bf16: three roundings on each side; fp32: sums of at most 600 terms a layer
    tol = 3 * 2.0 ** -8 if dtype == "bf16" else 600 * 2.0 ** -24
    assert np.abs(f64(y) - ref.numpy()).max() <= tol * ref.abs().max().item()


class Stem(torch.nn.Module):
    def __init__(self, kind, k, c=64):
        super().__init__()
        self.a = torch.nn.Conv2d(3, c, 3, 1, 1)
        self.pool = (torch.nn.MaxPool2d if kind == "max" else torch.nn.AvgPool2d)(*k)
        self.b = torch.nn.Conv2d(c, 64, 1)
        self.c = torch.nn.Conv2d(64, 16, 1)
        self.gap = torch.nn.AdaptiveAvgPool2d(1)

    def forward(self, x):
        return torch.flatten(self.gap(self.c(self.b(self.pool(self.a(x))))), 1)


@pytest.mark.parametrize("kind", ["max", "avg"])
@pytest.mark.parametrize("c", [64, 72])
@pytest.mark.parametrize("hw,k", [((16, 24), (3, 2, 1)), ((13, 72), (3, 2, 1)), ((15, 136), (3, 2, 1)),
                                  ((14, 14), (2, 2, 0))], ids=str)
def test_channels_last_pooling(kind, c, hw, k):
    """Pooling into channels-last (3 x 3, stride 2: 16 input columns per thread, 32 output columns per tile, 64
    channels per tile), and global average pooling out of it, against the same network in float64."""
    torch.manual_seed(hw[1])
    net = Stem(kind, k, c).to(torch.bfloat16).eval()
    x = torch.randn(2, 3, *hw).to(torch.bfloat16)
    say("channels-last pooling", kind, c, hw, k)
    model = cs.swap_backend(net.to(DEV), "implicit_gemm")
    y = model(x.to(DEV))
    torch.cuda.synchronize()
    assert "channels_last" in model.describe()
    ref = net.cpu().double()(x.double()).detach().numpy()
    # five bf16 roundings, averaged over the plane
    assert np.abs(f64(y) - ref).max() <= 5 * 2.0 ** -8 * np.abs(ref).max()


# N, C, H, W, K, R, stride, pad, dilation: single layers of the channels-last kernel.  Channels that fill their last
# 16-byte unit or not, rounded up to whole 128-byte pieces or not; a copy that needs two batches of images; planes of
# 8-, 4- and odd-pixel rows; the smallest work that takes this path.
LAYERS = [
    (3, 20, 15, 15, 24, 5, 1, 2, 1),
    (2, 60, 21, 20, 72, 3, 1, 1, 1),
    (2, 120, 16, 16, 64, 5, 2, 2, 1),
    (4, 48, 14, 14, 40, 3, 1, 2, 2),
    (1, 13, 33, 31, 17, 7, 2, 3, 1),
    (130, 128, 36, 36, 8, 5, 2, 2, 1),
    (7, 100, 33, 35, 72, 3, 1, 1, 1),
    (1, 31, 27, 27, 33, 3, 1, 0, 1),
    (1, 256, 14, 14, 64, 3, 1, 18, 18),       # dilation past the plane: taps past the whole buffer
]


@pytest.mark.parametrize("case", LAYERS, ids=str)
def test_channels_last_layer(case):
    N, C, H, W, K, R, st, pad, dil = case
    g = torch.Generator().manual_seed(C)
    x = torch.randn(N, C, H, W, generator=g).to(torch.bfloat16)
    w = (torch.randn(K, C, R, R, generator=g) / (C * R * R) ** 0.5).to(torch.bfloat16)
    b = torch.randn(K, generator=g).to(torch.bfloat16)
    say("channels-last layer", case)
    d = cs.describe(x.shape, w.shape, st, pad, dil, 1, torch.bfloat16, "implicit_gemm", True, True)
    assert "nhwc_conv_kernel" in d
    kw = dict(stride=st, padding=pad, dilation=dil, algo="implicit_gemm", relu=True)
    y = cs.conv2d(x.to(DEV), w.to(DEV), b.to(DEV), **kw)
    pk = cs.pack_filters(w.to(DEV), tuple(x.shape), bias=True, **kw)
    yp = cs.conv2d_prepacked(x.to(DEV), pk, tuple(w.shape), b.to(DEV), **kw)
    torch.cuda.synchronize()
    assert torch.equal(y, yp)
    ref = oracle.conv2d(f64(x), f64(w), f64(b), st, pad, dil, 1, True)
    # fp32 sums of C*R*R terms, then one bf16 rounding
    S = oracle.conv2d(np.abs(f64(x)), np.abs(f64(w)), np.abs(f64(b)), st, pad, dil, 1, False)
    assert (np.abs(f64(y) - ref) <= (C * R * R + 1) * 2.0 ** -24 * S + 2.0 ** -8 * np.abs(ref) + 1e-30).all()
    # never more workspace than the static scratch holds
    assert cs._lib.workspace_bytes(cs._lib.make_desc(N, C, H, W, K, R, R, st, pad, dil, 1, "bf16", True, True),
                                   "implicit_gemm") <= cs._lib.static_scratch_capacity()


class Inverted(torch.nn.Module):
    def __init__(self, c, mid, k, st, pad, res, more):
        super().__init__()
        self.a = torch.nn.Conv2d(c, mid, 1)
        self.b = torch.nn.Conv2d(mid, mid, 3, st, pad, groups=mid)
        self.c = torch.nn.Conv2d(mid, k, 1)
        self.d = torch.nn.Conv2d(k, 20, 1)
        self.res, self.more = res, more

    def forward(self, x):
        y = self.c(torch.relu(self.b(torch.relu(self.a(x)))))
        if self.res:
            y = y + x
        return self.d(y) if self.more else y


# N, C, mid, K, H, W, stride, pad, residual, further layer.  Depthwise strips of 2 x 4 and 2 x 7 (stride 1), 1 x 4 and
# 1 x 7 (stride 2) outputs with remainders, no padding and padding 2, one-row planes; float32 layers channels-last.
INVERTED = [
    (2, 16, 40, 16, 7, 9, 1, 1, True, False),
    (1, 8, 24, 16, 8, 5, 2, 1, False, True),
    (3, 24, 72, 40, 13, 14, 2, 0, False, False),
    (2, 32, 64, 32, 6, 11, 1, 2, False, True),
    (1, 64, 200, 64, 4, 3, 1, 0, False, False),
    (40, 32, 192, 32, 14, 14, 1, 1, True, False),
    (70, 96, 576, 96, 7, 7, 1, 1, True, True),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", INVERTED, ids=str)
def test_channels_last_depthwise(case, dtype):
    N, C, mid, K, H, W, st, pad, res, more = case
    torch.manual_seed(mid)
    net = Inverted(C, mid, K, st, pad, res, more).to(TDT[dtype]).eval()
    x = torch.randn(N, C, H, W).to(TDT[dtype])
    model = cs.swap_backend(net.to(DEV), {"a": "implicit_gemm", "b": "direct", "c": "implicit_gemm",
                                          "d": "implicit_gemm"})
    say("channels-last depthwise", case, dtype)
    y = model(x.to(DEV))
    torch.cuda.synchronize()
    assert model.describe().count("channels_last") >= 3
    ref = net.cpu().double()(x.double()).detach().numpy()
    # fp32: sums of at most 600 terms a layer; bf16: one rounding per layer and the add
    tol = 600 * 2.0 ** -24 if dtype == "f32" else 4 * 2.0 ** -8
    assert np.abs(f64(y) - ref).max() <= tol * np.abs(ref).max()
