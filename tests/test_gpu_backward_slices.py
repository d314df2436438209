"""Backward pass: the forms of the activation side of wgrad_kernel (a dword of four channels per pixel, or a
byte) on tiles, channel counts and pixel counts with remainders, and layers whose contractions are cut into
one, few and many slices.  Against the float64 oracle with the bounds of tests/test_gpu_backward.py."""

import numpy as np
import pytest
import torch

from paper_2002_09481_amd import binding as ax
from paper_2002_09481_amd import inputs as I

import test_gpu_backward as B

pytestmark = pytest.mark.gpu

# N, H, W, Cin, KH, KW, Cout, stride, pad, dilation
SHAPES = [
    (1, 5, 7, 4, 1, 1, 3, 1, 0, 1),        # one dword of channels, one stage, fewer taps than a tile
    (2, 9, 11, 36, 3, 3, 130, 1, 1, 1),    # 324 taps: a second, ragged tap tile of 256; ragged channel tile
    (2, 9, 11, 35, 3, 3, 130, 1, 1, 1),    # the same, byte loads
    (1, 33, 31, 44, 1, 1, 66, 1, 0, 1),    # 128 x 128 tiles, ragged stage of 1023 pixels
    (3, 10, 10, 20, 3, 3, 40, 2, 1, 1),    # 128 x 64 tiles, classes of a stride
    (1, 3, 3, 512, 3, 3, 160, 1, 1, 1),    # nine pixels, 144 stages of the input gradient
    (16, 24, 24, 8, 3, 3, 16, 1, 1, 2),    # many pixels, few taps: many slices; dilation
    (1, 46, 46, 4, 1, 1, 5280, 45, 0, 1),  # 2025 classes of a stride, 165 stages: a launch holds 32 slices of them
]


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_gradients_match_the_oracle(shape, signed):
    B._check(shape, sum(shape) + signed, signed, gy_kind="wide" if signed else "normal")


def test_activations_at_any_byte():
    """The dword form needs x at a multiple of four bytes: a view one byte on takes the byte form, same gradients."""
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    n = 2 * 9 * 11 * 36
    buf = torch.randint(0, 256, (n + 8,), generator=g, device="cuda", dtype=torch.uint8)
    x = buf[:n].view(2, 9, 11, 36)
    y = torch.empty(n + 8, device="cuda", dtype=torch.uint8)
    y[1:n + 1] = buf[:n]
    w = torch.randint(0, 256, (3, 3, 36, 40), generator=g, device="cuda", dtype=torch.uint8)
    gy = torch.randn((2, 9, 11, 40), generator=g, device="cuda")
    q = I.Quant(0.02, 3, 0.01, 128, None)
    a = ax.ax_conv2d_backward(x, w, gy, 1, 1, q)
    b = ax.ax_conv2d_backward(y[1:n + 1].view(2, 9, 11, 36), w, gy, 1, 1, q)
    torch.cuda.synchronize()
    for p, r in zip(b, a):
        assert torch.equal(p, r)
    assert all(np.isfinite(t.cpu().numpy()).all() for t in a)
