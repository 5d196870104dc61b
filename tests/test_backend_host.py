"""Host-side checks of the model executor: lowering of traced networks,
batch-norm folding, the arena plan (no two simultaneously live values share
bytes) and argument errors.  No kernel is launched: planning is host-only
and the filter pointers are never read before binding."""
import itertools

import numpy as np
import pytest
import torch
from torch import nn

import oracle
import paper_2410_08300_amd as cs
from paper_2410_08300_amd import _lib, backend
import variants
from nets import ConvStack, ResNetSmall, SharedFlatten, randomize_bn


def test_listing1_lowering_and_plan():
    m = cs.swap_backend(ConvStack(), ["direct", "smm"])
    assert m.ops == [("conv", "0"), ("maxpool", "2"), ("conv", "3"), ("flatten", "_5")]
    nbytes = m._native.plan(2, 3, 32, 32)
    assert m._native.output_shape() == (2, 32 * 16 * 16)
    d = m._native.describe()
    assert "0 conv v0 -> v1 [2 16 32 32] algo=direct relu" in d
    assert "2 conv v2 -> v3 [2 32 16 16] algo=smm relu offset=-1" in d   # writes the caller's output
    assert nbytes > 0


def test_residual_net_lowering_fuses_and_folds():
    torch.manual_seed(0)
    net = randomize_bn(ResNetSmall(), 1)
    m = cs.swap_backend(net, "default")
    kinds = [k for k, _ in m.ops]
    # BN folded (no bn ops), ReLUs fused (no relu ops), dropout dropped
    assert kinds == ["conv", "maxpool", "conv", "conv", "add", "conv", "conv", "conv", "add", "avgpool",
                     "global_avgpool", "flatten", "linear"]
    nbytes = m._native.plan(3, 3, 64, 64)
    assert m._native.output_shape() == (3, 10)
    d = m._native.describe().splitlines()
    assert d[0].startswith("0 conv v0 -> v1 [3 16 32 32]") and d[0].split()[-2] == "relu"
    assert "add v" in d[4] and " relu " in d[4] + " "
    # Both residual adds are fused into the epilogue of the convolution that
    # produces one operand; that convolution reads the other operand and takes
    # over the add's ReLU, and the add's output is the convolution's output.
    fused = [line for line in d if " add " in " " + line]
    assert len(fused) == 2 and all(line.split()[-2] == "fused" for line in fused)
    for line in fused:
        toks = line.split()
        a, b = int(toks[2][1:]), int(toks[4][1:])
        convs = [c for c in d if c.split()[1] == "conv" and c.split()[4] in ("v%d" % a, "v%d" % b)
                 and " + v" in c]
        assert len(convs) == 1
        ctoks = convs[0].split()
        x = int(ctoks[4][1:])
        y = b if x == a else a
        assert ctoks[ctoks.index("+") + 1] == "v%d" % y and ctoks[ctoks.index("+") + 2] == "relu"
    # Arena plan: values live at the same time never share bytes, all within
    # the arena, 256-byte aligned.  A fused add's output is stored where the
    # convolution's output is, so its reads extend that value's lifetime.
    reads, prod, alias = [], {}, {}
    for i, line in enumerate(d[:-1]):
        toks = line.split()
        ins = [int(t[1:]) for t in toks[2:toks.index("->")] if t.startswith("v")]
        out = int(toks[toks.index("->") + 1][1:])
        reads.append(ins)
        prod[out] = i
        if toks[-2] == "fused":
            alias[out] = [v for v in ins if "+ v" in d[prod[v]]][0]
    last = dict(prod)
    for i, ins in enumerate(reads):
        for v in ins:
            r = alias.get(v, v)
            last[r] = max(last.get(r, -1), i)
    place = {}
    for v in prod:
        off, nb = m._native.placement(v)
        if off >= 0:
            place[v] = (off, nb)
            assert off % 256 == 0 and off + nb <= nbytes
    # flatten's output shares its input's storage
    fl = [i for i, (k, _) in enumerate(m.ops) if k == "flatten"][0]
    assert m._native.placement(fl + 1)[0] == m._native.placement(fl)[0]
    for v, x in alias.items():
        assert place[v] == place[x]
    roots = {v: p for v, p in place.items() if m.ops[prod[v]][0] != "flatten" and v not in alias}
    for a, b in itertools.combinations(roots, 2):
        la, lb = (prod[a], last[a]), (prod[b], last[b])
        if la[0] <= lb[1] and lb[0] <= la[1]:
            (oa, na), (ob, nb2) = roots[a], roots[b]
            assert oa + na <= ob or ob + nb2 <= oa, (a, b)
    # some reuse happened: the activation region is smaller than the sum of the values
    lo = min(o for o, _ in roots.values())
    hi = max(o + nb for o, nb in roots.values())
    assert sum(nb for _, nb in roots.values()) > hi - lo


def test_bn_fold_matches_conv_then_bn():
    torch.manual_seed(2)
    conv = nn.Conv2d(5, 7, 3, 2, 1, bias=True).double()
    bn = randomize_bn(nn.Sequential(nn.BatchNorm2d(7)), 3)[0].double()
    x = torch.randn(2, 5, 9, 8, dtype=torch.float64)
    ref = bn(conv(x)).detach().numpy()
    w, b = backend._fold_bn(conv, bn)
    got = oracle.conv2d(x.numpy(), w.numpy(), b.numpy(), 2, 1)
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))


def test_unsupported_nodes_and_errors():
    class Sig(nn.Module):
        def __init__(self):
            super().__init__()
            self.c = nn.Conv2d(3, 4, 3)

        def forward(self, x):
            return torch.sigmoid(self.c(x))

    with pytest.raises(NotImplementedError):
        cs.swap_backend(Sig())
    with pytest.raises(NotImplementedError):
        cs.swap_backend(nn.Sequential(nn.Conv2d(3, 4, 3), nn.ReLU(), nn.BatchNorm2d(4)))   # BN not after a conv
    with pytest.raises(ValueError):
        cs.swap_backend(ConvStack(), ["direct"])                                            # list length
    with pytest.raises(ValueError):
        cs.swap_backend(ConvStack(), "torch")
    m = cs.swap_backend(ConvStack())
    with pytest.raises(_lib.Conv2dError):
        m._native.plan(2, 4, 32, 32)                  # 4 input channels, conv1 expects 3
    with pytest.raises(_lib.Conv2dError):
        m._native.forward(1 << 20, 2 << 20, None)     # not bound
    with pytest.raises(_lib.Conv2dError):
        m._native.plan(2, 3, 1, 1)                    # the 2x2 pool has no output
    nm = _lib.NativeModel("f32")
    with pytest.raises(_lib.Conv2dError):
        nm.plan(1, 3, 8, 8)                           # no output set
    with pytest.raises(_lib.Conv2dError):
        nm.relu(5)                                    # no such value
    v = nm.flatten(0)
    nm.set_output(v)
    with pytest.raises(_lib.Conv2dError):
        nm.plan(1, 3, 8, 8)                           # the output is the input itself
    with pytest.raises(ValueError):
        m(torch.randn(2, 3, 32, 32))                  # CPU input


def test_library_exports_model_functions():
    import os
    import re
    hdr = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "convsel_model.h")
    text = re.sub(r"/\*.*?\*/", "", open(hdr).read(), flags=re.S)
    names = sorted(set(re.findall(r"\b(convsel_model_[a-z_]+)\s*\(", text)))
    assert names == sorted(_lib.EXPORTED_MODEL)
    L = _lib.lib()
    for n in names:
        assert hasattr(L, n), n


def _lowered(net, shape):
    m = cs.swap_backend(net, "implicit_gemm")
    m._native.plan(*shape)
    return m._native.describe().splitlines()[:-1]


def test_residual_fusion_only_where_it_is_exact():
    """An add goes into a convolution's epilogue only when that is the same
    computation: the convolution's output is read by nothing else, the
    convolution has no ReLU of its own, and the other operand already
    exists when the convolution runs."""
    class Twice(nn.Module):          # conv output read twice: by the add and by the output add
        def __init__(self):
            super().__init__()
            self.c = nn.Conv2d(8, 8, 3, 1, 1)

        def forward(self, x):
            y = self.c(x)
            return (y + x) + y

    class Relu(nn.Module):           # the conv's own ReLU comes before the add
        def __init__(self):
            super().__init__()
            self.c = nn.Conv2d(8, 8, 3, 1, 1)

        def forward(self, x):
            return torch.relu(self.c(x)) + x

    class Later(nn.Module):          # the other operand is computed after the conv
        def __init__(self):
            super().__init__()
            self.a = nn.Conv2d(8, 8, 3, 1, 1)
            self.b = nn.Conv2d(8, 8, 1)

        def forward(self, x):
            y = self.a(x)
            z = self.b(x)
            return y + z

    class Self(nn.Module):           # y + y
        def __init__(self):
            super().__init__()
            self.c = nn.Conv2d(8, 8, 3, 1, 1)

        def forward(self, x):
            y = self.c(x)
            return y + y

    class Plain(nn.Module):          # fused: conv(x) + x, then ReLU
        def __init__(self):
            super().__init__()
            self.c = nn.Conv2d(8, 8, 3, 1, 1)

        def forward(self, x):
            return torch.relu(self.c(x) + x)

    shape = (2, 8, 6, 6)
    for net in (Twice(), Relu(), Self()):
        d = _lowered(net, shape)
        assert not any(" fused" in line for line in d), (type(net).__name__, d)
        assert not any(" + v" in line for line in d if " conv " in line)
    d = _lowered(Later(), shape)
    # b runs after a, so a cannot take z as its residual, but b can take a's output
    conv_b = [line for line in d if line.startswith("1 conv")][0]
    assert " + v1" in conv_b and any(line.split()[1] == "add" and " fused" in line for line in d)
    d = _lowered(Plain(), shape)
    assert d[0].startswith("0 conv v0 -> v1") and " + v0 relu " in d[0] + " " and d[1].endswith("fused offset=-1")


def test_channels_last_plan():
    """bf16 implicit GEMM chains are planned channels-last; the copy of the
    model's input that the first convolution then reads lies inside the
    arena, apart from every value and package that is live with it."""
    net = nn.Sequential(nn.Conv2d(64, 16, 1), nn.ReLU(), nn.Conv2d(16, 16, 3, 1, 1), nn.ReLU(),
                        nn.Conv2d(16, 64, 1)).to(torch.bfloat16)
    m = cs.swap_backend(net, "implicit_gemm")
    nbytes = m._native.plan(8, 64, 28, 28)
    d = m._native.describe().splitlines()
    assert sum("channels_last" in line for line in d) == 3
    copy = int(d[0].split("copy@")[1].split()[0])
    size = 8 * 64 * 28 * 28 * 2
    ws = int(d[-1].split("@")[1])
    assert copy >= ws and copy + size <= nbytes
    off, nb = m._native.placement(1)               # conv1's output: written while the copy is read
    assert off + nb <= copy or copy + size <= off
    # a lone convolution keeps its own kernels, and so does a float32 model
    lone = cs.swap_backend(nn.Sequential(nn.Conv2d(64, 16, 3)).to(torch.bfloat16), "implicit_gemm")
    lone._native.plan(2, 64, 14, 14)
    assert "channels_last" not in lone._native.describe()
    f32 = cs.swap_backend(nn.Sequential(nn.Conv2d(64, 16, 1), nn.Conv2d(16, 64, 1)), "implicit_gemm")
    f32._native.plan(2, 64, 14, 14)
    assert "channels_last" not in f32._native.describe()


@pytest.mark.parametrize("pooled", [True, False])
def test_flattened_value_is_not_read_from_a_channels_last_copy(pooled):
    """A linear layer reads a flattened image in place, also where the image has a channels-last copy."""
    m = cs.swap_backend(SharedFlatten(pooled).to(torch.bfloat16), "implicit_gemm")
    m._native.plan(2, 64, 14 if pooled else 7, 14 if pooled else 7)
    d = m._native.describe().splitlines()
    assert [line.split()[1] for line in d if "copy@" in line] == ["conv"]
    assert sum(line.split()[1] == "linear" for line in d) == 2


@pytest.mark.parametrize("stride,size,algo", [(2, 224, "implicit_gemm"), (4, 300, "implicit_precomp_gemm")])
def test_default_choice_of_a_stem(stride, size, algo):
    """A model's stride 2 stem of filter rows runs implicit GEMM by default; other layers keep the library's choice."""
    net = nn.Sequential(nn.Conv2d(3, 64, 7, stride, 3)).to(torch.bfloat16)
    m = cs.swap_backend(net)
    m._native.plan(4, 3, size, size)
    desc = _lib.make_desc(4, 3, size, size, 64, 7, 7, stride, 3, 1, 1, "bf16", True)
    assert _lib.default_algo(desc) == "implicit_precomp_gemm"
    assert "algo=%s" % algo in m._native.describe()


# C, H, W, R, pad, dilation, N: bf16 layers of the channels-last kernel, whose input buffer holds N*H*W pixels behind
# pad rows and columns.
@pytest.mark.parametrize("case", [(256, 14, 14, 3, 18, 18, 1), (256, 14, 14, 3, 18, 18, 2), (256, 14, 14, 3, 13, 13, 1),
                                  (2048, 7, 7, 3, 12, 12, 1), (256, 14, 14, 3, 14, 14, 1), (512, 3, 4, 7, 3, 1, 1),
                                  (512, 4, 3, 7, 3, 1, 1), (64, 28, 28, 5, 2, 1, 4), (64, 9, 30, 5, 16, 8, 1)], ids=str)
def test_scalar_tap_offsets_stay_within_the_buffer(case):
    C, H, W, R, pad, dil, N = case
    d = cs.describe((N, C, H, W), (256, C, R, R), 1, pad, dil, 1, torch.bfloat16, "implicit_gemm")
    assert "nhwc_conv_kernel" in d
    pixel = 2 * C
    last_tap = ((R - 1) * dil * W + (R - 1) * dil) * pixel + pixel - 128     # its last 128-byte piece
    inside = last_tap <= (N * H * W + pad * W + pad) * pixel
    assert ("taps=uniform" if inside else "taps=per_lane") in d


class OutputReadAgain(nn.Module):
    """The model's output value is also read by a layer whose result is not used."""

    def __init__(self, pool):
        super().__init__()
        self.a, self.b = nn.Conv2d(16, 32, 1), nn.Conv2d(32, 16, 1)
        self.last = nn.AdaptiveAvgPool2d(1) if pool == "gap" else nn.MaxPool2d(7)
        self.fc = nn.Linear(16, 8)

    def forward(self, x):
        y = torch.flatten(self.last(self.b(self.a(x))), 1)
        self.fc(y)
        return y


@pytest.mark.parametrize("pool", ["gap", "max"])
def test_layers_that_read_the_output_tensor_do_not_assume_its_alignment(pool):
    """The channels-last kernel reads 16-byte units in place: of values in the arena only."""
    m = cs.swap_backend(OutputReadAgain(pool).to(torch.bfloat16), "implicit_gemm")
    m._native.plan(2, 16, 7, 7)
    d = m._native.describe().splitlines()
    assert sum("channels_last" in line for line in d) == 2
    assert not any("channels_last" in line for line in d if line.split()[1] == "linear")


def test_variant_cases_cover_what_is_dispatched():
    """Every variant of the channels-last convolution that random shapes reach is reached by a case of variants.py
    (whose results the GPU tests check), in each dtype, tile, tap form and output layout."""
    covered = set()
    for case in variants.CASES:
        m = variants.lower(case, variants.Pair(*case))
        m._native.plan(*case[1:5])
        covered |= variants.reached(case, m._native.describe())
    tiles = {v[:5] for v in covered}
    bf16 = {("128x128", "2", "1"), ("64x128", "3", "1"), ("64x128", "2", "1"), ("64x64", "4", "1"), ("64x64", "2", "1"),
            ("32x32", "8", "1"), ("32x32", "4", "4")}
    assert {v[1:4] for v in tiles if v[0] == "bf16"} == bf16
    assert len({v for v in tiles if v[0] == "bf16"}) == 2 * len(bf16)
    rng = np.random.default_rng(1)
    seen, plans = set(), 0

    def size(lo, hi):
        return int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))

    while plans < 3000:
        dtype = "bf16" if rng.random() < 0.6 else "f32"
        unit = 8 if dtype == "bf16" else 4
        n, c, k, k2 = size(1, 128), size(1, 60) * unit, size(1, 60) * unit, size(1, 60) * unit
        c, k = (8 * v if rng.random() < 0.4 else v for v in (c, k))
        r, r2, h, stride = rng.choice((1, 1, 3, 5)), rng.choice((1, 1, 3)), size(3, 60), rng.choice((1, 1, 2))
        m = _lib.NativeModel(dtype)
        case = (dtype, n, c, h, h + 1, k, int(r), int(stride), int(r) // 2, 1, k2, int(r2))
        v = m.conv(0, c, k, r, r, (stride, stride), (r // 2, r // 2), (1, 1), 1, "implicit_gemm", 256, 256, True)
        if dtype == "f32":
            v = m.conv(v, k, k, 3, 3, (1, 1), (1, 1), (1, 1), k, "direct", 256, 256, True)
        v = m.conv(v, k, k2, r2, r2, (1, 1), (r2 // 2, r2 // 2), (1, 1), 1, "implicit_gemm", 256, 256, True)
        m.set_output(v)
        try:
            m.plan(n, c, h, h + 1)
        except _lib.Conv2dError:
            continue
        seen |= variants.reached(case, m.describe())
        plans += 1
    assert len(seen) > 60 and seen <= covered, sorted(seen - covered)


class TwoChains(nn.Module):
    """Two pairs of convolutions with a layer between them that channels-last values do not pass."""

    def __init__(self, first, second, c):
        super().__init__()
        self.first, self.between, self.second = first, nn.Conv2d(c, c, 3, 1, 1), second

    def forward(self, x):
        return self.second(self.between(self.first(x)))


def _pair(c, depthwise):
    mid = [nn.Conv2d(c, c, 3, 1, 1, groups=c)] if depthwise else []
    return nn.Sequential(nn.Conv2d(c, c, 1), *mid, nn.Conv2d(c, c, 1))


def _chains_of(net, shape):
    algo = {name: "direct" if m.groups > 1 else "implicit_gemm" for name, m in net.named_modules()
            if isinstance(m, nn.Conv2d)}
    algo["between"] = "im2col_gemm"
    m = cs.swap_backend(net, algo)
    m._native.plan(*shape)
    return ["channels_last" in line for line in m._native.describe().splitlines() if " conv " in " " + line]


def test_layouts_are_decided_chain_by_chain():
    """bf16: an odd plane, or a depthwise layer, decides for the convolutions it is connected to, and no others."""
    net = TwoChains(nn.Sequential(nn.Conv2d(64, 64, 1), nn.Conv2d(64, 64, 3, 1, 1, groups=64), nn.Conv2d(64, 64, 1),
                                  nn.MaxPool2d(3, 1)), _pair(64, False), 64).to(torch.bfloat16)
    assert _chains_of(net, (40, 64, 58, 58)) == [True] * 3 + [False] * 3      # then 56 x 56: whole planes, large copies
    net = TwoChains(_pair(32, True), _pair(32, False), 32)                   # float32: all of them
    assert _chains_of(net, (2, 32, 14, 14)) == [True] * 3 + [False] + [True] * 2
    net = TwoChains(nn.Sequential(nn.Conv2d(64, 64, 1), nn.Conv2d(64, 64, 3, 2, 1)), _pair(64, False), 64)
    net = net.to(torch.bfloat16)
    assert _chains_of(net, (40, 64, 56, 56)) == [False] * 5       # 28 x 28: whole planes, large copies
    assert _chains_of(net, (40, 64, 54, 54)) == [True] * 2 + [False] + [True] * 2   # 27 x 27


def test_a_copy_counts_once_for_all_its_readers():
    """1.6 MB read by two convolutions is a small copy, although its readers read 3.2 MB."""

    class Fork(nn.Module):
        def __init__(self):
            super().__init__()
            self.a, self.b, self.c = (nn.Conv2d(i, o, 1) for i, o in ((64, 32), (64, 32), (32, 64)))

        def forward(self, x):
            return self.c(self.a(x) + self.b(x))

    m = cs.swap_backend(Fork().to(torch.bfloat16), "implicit_gemm")
    m._native.plan(16, 64, 28, 28)
    assert m._native.describe().count("channels_last") == 3


@pytest.mark.parametrize("dtype,width,expected", [("bf16", 56, 0), ("bf16", 60, 3), ("bf16", 14, 3), ("f32", 56, 3)])
def test_depthwise_chains_by_row_width(dtype, width, expected):
    """bf16 depthwise layers on rows of whole 16 bytes are as fast on planes."""
    net = nn.Sequential(nn.Conv2d(24, 144, 1), nn.Conv2d(144, 144, 3, 1, 1, groups=144), nn.Conv2d(144, 24, 1))
    m = cs.swap_backend(net.to(variants.DTYPES[dtype]), ["implicit_gemm", "direct", "implicit_gemm"])
    m._native.plan(8, 24, width, width)
    assert m._native.describe().count("channels_last") == expected


@pytest.mark.parametrize("images,expected", [((1 << 24) - 1, 3), (1 << 24, 0)])
def test_copies_of_more_workgroups_than_a_grid_holds_stay_planes(images, expected):
    """One workgroup of 256 threads copies an image of up to 64 pixels; a grid has fewer than 2^32 threads."""
    net = nn.Sequential(nn.Conv2d(8, 8, 1), nn.Conv2d(8, 8, 3, 1, 1, groups=8), nn.Conv2d(8, 8, 1))
    m = cs.swap_backend(net.to(torch.bfloat16), ["implicit_gemm", "direct", "implicit_gemm"])
    m._native.plan(images, 8, 2, 1)
    assert m._native.describe().count("channels_last") == expected
