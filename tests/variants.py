"""Shapes that reach every variant of the channels-last convolution: a convolution of C -> K channels, R x R, that
writes channels-last, a depthwise 3 x 3 layer in fp32 (whose chains are channels-last around one only), and a
convolution K -> K2, R2 x R2, that writes planes (and adds the input to them where the shapes are equal)."""
import re

import torch
from torch import nn

import paper_2410_08300_amd as cs

# dtype, N, C, H, W, K, R, stride, pad, dilation, K2, R2
CASES = [
    ("bf16", 1, 8, 3, 3, 128, 1, 1, 0, 1, 8, 3),
    ("bf16", 1, 8, 3, 4, 64, 3, 2, 1, 1, 16, 3),
    ("bf16", 1, 8, 4, 5, 8, 1, 2, 0, 1, 8, 1),
    ("bf16", 1, 16, 3, 3, 48, 5, 2, 2, 1, 16, 3),
    ("bf16", 1, 16, 3, 5, 72, 1, 2, 0, 1, 24, 3),
    ("bf16", 1, 16, 4, 5, 64, 1, 2, 0, 1, 24, 1),
    ("bf16", 1, 16, 4, 6, 16, 1, 1, 0, 1, 16, 1),
    ("bf16", 1, 16, 7, 8, 64, 1, 2, 0, 1, 8, 1),
    ("bf16", 1, 64, 3, 3, 8, 1, 2, 0, 1, 32, 1),
    ("bf16", 1, 64, 4, 4, 64, 3, 2, 2, 2, 16, 1),
    ("bf16", 2, 8, 4, 4, 64, 1, 1, 0, 1, 8, 3),
    ("bf16", 2, 24, 7, 8, 48, 1, 2, 0, 1, 16, 3),
    ("bf16", 6, 8, 56, 58, 64, 1, 1, 0, 1, 24, 1),
    ("bf16", 6, 32, 53, 52, 8, 1, 1, 0, 1, 8, 1),
    ("bf16", 7, 64, 36, 37, 8, 1, 1, 0, 1, 8, 1),
    ("bf16", 11, 64, 51, 51, 8, 1, 1, 0, 1, 8, 3),
    ("bf16", 13, 24, 57, 58, 8, 1, 1, 0, 1, 80, 1),
    ("bf16", 15, 8, 43, 42, 192, 1, 1, 0, 1, 208, 1),
    ("bf16", 15, 16, 37, 36, 64, 1, 1, 0, 1, 16, 1),
    ("bf16", 17, 8, 13, 14, 64, 1, 1, 0, 1, 72, 1),
    ("bf16", 17, 16, 50, 49, 64, 1, 1, 0, 1, 72, 1),
    ("bf16", 18, 184, 53, 52, 16, 1, 1, 0, 1, 104, 3),
    ("bf16", 18, 184, 59, 61, 72, 1, 1, 0, 1, 128, 1),
    ("bf16", 20, 16, 45, 46, 128, 1, 1, 0, 1, 8, 1),
    ("bf16", 20, 32, 23, 22, 256, 1, 1, 0, 1, 264, 1),
    ("bf16", 21, 16, 11, 12, 64, 1, 2, 0, 1, 328, 1),
    ("bf16", 23, 8, 20, 20, 64, 1, 1, 0, 1, 8, 1),
    ("bf16", 24, 8, 26, 27, 8, 1, 1, 0, 1, 8, 1),
    ("bf16", 24, 16, 48, 50, 128, 1, 1, 0, 1, 72, 1),
    ("bf16", 32, 40, 19, 20, 8, 1, 1, 0, 1, 392, 1),
    ("bf16", 34, 128, 42, 42, 128, 1, 1, 0, 1, 112, 1),
    ("bf16", 36, 256, 39, 38, 256, 1, 2, 0, 1, 208, 1),
    ("bf16", 39, 8, 41, 40, 8, 1, 1, 0, 1, 88, 3),
    ("bf16", 45, 64, 51, 51, 208, 1, 2, 0, 1, 72, 1),
    ("bf16", 46, 8, 16, 16, 8, 5, 1, 4, 2, 424, 1),
    ("bf16", 46, 16, 24, 23, 256, 1, 1, 0, 1, 72, 1),
    ("bf16", 54, 16, 16, 15, 200, 5, 1, 2, 1, 224, 1),
    ("bf16", 54, 56, 21, 22, 32, 1, 1, 0, 1, 72, 3),
    ("bf16", 65, 16, 51, 52, 64, 1, 2, 0, 1, 96, 1),
    ("bf16", 70, 16, 16, 16, 8, 1, 1, 0, 1, 8, 1),
    ("bf16", 89, 16, 30, 31, 64, 1, 2, 0, 1, 224, 1),
    ("bf16", 116, 16, 9, 8, 8, 1, 1, 0, 1, 8, 1),
    ("f32", 1, 4, 3, 3, 64, 1, 2, 0, 1, 12, 1),
    ("f32", 1, 4, 4, 4, 4, 3, 2, 2, 2, 4, 3),
    ("f32", 1, 4, 5, 5, 32, 1, 2, 0, 1, 4, 3),
    ("f32", 1, 32, 3, 3, 12, 1, 1, 0, 1, 4, 1),
    ("f32", 16, 8, 38, 38, 8, 1, 1, 0, 1, 200, 1),
    ("f32", 16, 32, 23, 23, 4, 1, 1, 0, 1, 12, 1),
    ("f32", 23, 4, 20, 21, 32, 1, 1, 0, 1, 4, 1),
    ("f32", 32, 8, 37, 39, 96, 1, 1, 0, 1, 16, 1),
    ("f32", 38, 32, 34, 33, 4, 1, 1, 0, 1, 80, 1),
    ("f32", 53, 4, 20, 19, 4, 1, 1, 0, 1, 4, 1),
    ("f32", 65, 4, 14, 16, 4, 1, 1, 0, 1, 4, 1),
    ("f32", 77, 32, 48, 48, 96, 1, 2, 0, 1, 84, 1),
    ("f32", 79, 16, 45, 45, 32, 1, 2, 0, 1, 84, 1),
    ("f32", 86, 4, 15, 16, 32, 1, 1, 0, 1, 4, 1),
    ("f32", 101, 4, 9, 10, 32, 1, 1, 0, 1, 4, 1),
    ("f32", 120, 32, 13, 13, 4, 1, 1, 0, 1, 8, 1),
    # the input added to planes of 8-, 4- and odd-pixel rows
    ("bf16", 18, 64, 28, 28, 72, 1, 1, 0, 1, 64, 3),
    ("bf16", 24, 64, 26, 26, 72, 1, 1, 0, 1, 64, 3),
    ("bf16", 24, 64, 27, 27, 72, 1, 1, 0, 1, 64, 3),
    ("bf16", 60, 128, 27, 27, 72, 1, 1, 0, 1, 128, 3),
    ("bf16", 3, 64, 9, 9, 72, 1, 1, 0, 1, 64, 1),
    ("f32", 24, 64, 14, 14, 64, 1, 1, 0, 1, 64, 1),
    ("f32", 40, 64, 13, 13, 64, 1, 1, 0, 1, 64, 1),
]
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


class Pair(nn.Module):
    def __init__(self, dtype, n, c, h, w, k, r, stride, pad, dil, k2, r2):
        super().__init__()
        self.a = nn.Conv2d(c, k, r, stride, pad, dil)
        self.dw = nn.Conv2d(k, k, 3, 1, 1, groups=k) if dtype == "f32" else None
        self.b = nn.Conv2d(k, k2, r2, 1, r2 // 2)
        self.res = stride == 1 and c == k2 and 2 * pad == dil * (r - 1)
        self.to(DTYPES[dtype])

    def forward(self, x):
        y = torch.relu(self.a(x))
        if self.dw is not None:
            y = torch.relu(self.dw(y))
        y = self.b(y)
        return torch.relu(y + x) if self.res else y


def lower(case, net):
    return cs.swap_backend(net, {"a": "implicit_gemm", "dw": "direct", "b": "implicit_gemm"})


def reached(case, description):
    """The variants of a described plan: dtype, tile, stages, wave groups, tap form, output layout, and for planes
    the whole pixels their rows divide into (8, 4 or 1)."""
    dtype, n, c, h, w, k, r, stride, pad, dil, k2, r2 = case
    p, q = ((v + 2 * pad - dil * (r - 1) - 1) // stride + 1 for v in (h, w))
    unit = 1 if p * q % 4 else 4 if p * q % 8 or dtype == "f32" else 8
    found = re.findall(r"tile=(\S+) stages=(\d) groups=(\d) taps=(\S+) out=(\S+)", description)
    return {(dtype,) + v + (unit if v[4] == "planes" else 0,) for v in found}
