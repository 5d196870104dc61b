"""Kernel variants at the sizes where their tiling can go wrong: tile edges,
remainders, and the smallest and largest shapes of each dispatch rule."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_08300_amd as cs
from gpu_util import f64, say

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TDT = {"f32": torch.float32, "bf16": torch.bfloat16}


# N, C, H, W, R, S, stride, pad, dilation, groups.  The LDS gather's tiles are 64 output columns and
# 64 (bf16) or 32 (fp32) channels; rows that are no whole units and very long or wide filters keep the others.
IM2COL = [
    (2, 64, 5, 65, 3, 3, 1, 1, 1, 1),         # one column past a column tile
    (1, 72, 9, 64, 3, 3, 1, 1, 1, 1),         # channel remainder of 8, one full column tile
    (2, 200, 7, 7, 3, 3, 2, 1, 1, 2),         # groups with a channel remainder, stride 2
    (1, 8, 130, 3, 1, 1, 1, 0, 1, 1),         # one tap, narrow rows
    (2, 64, 1, 1, 1, 1, 1, 0, 1, 1),          # one pixel: one staged row and column
    (1, 96, 13, 150, 5, 3, (1, 2), (2, 1), 1, 1),  # mixed strides, 75 columns
    (1, 16, 20, 21, 7, 7, 1, 3, 1, 1),        # 49 taps: smaller channel chunks
    (1, 8, 40, 40, 17, 17, 1, 8, 1, 1),       # 289 units per pixel: the general vector gather
    (1, 16, 150, 150, 3, 3, 1, 60, 60, 1),    # dilation 60: tiles halved until they fit, or the vector gather
    (3, 3, 17, 18, 7, 7, 2, 3, 1, 1),         # 147 elements per row: the element gather
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
