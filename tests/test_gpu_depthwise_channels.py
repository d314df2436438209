"""3 x 3 depthwise layers against the oracle where a thread's walk over the items can go wrong: channel
groups that do not divide the number of threads, images smaller than one step of the walk (its carries
from column to row to image), strides, dilation and outputs that are not 16-byte aligned.  WALK holds the
layers whose threads come round at least twice (two items of four channels per round)."""

import numpy as np
import pytest
import torch

from gpu_common import assert_parity, to_dev
from oracle import oracle
from paper_2002_09481_amd import binding as ax
from paper_2002_09481_amd import inputs as I

pytestmark = pytest.mark.gpu

# N, H, W, C, stride, pad, dilation: over 4e6 lookups each, so that the table is kept in LDS
CASES = [(3, 57, 55, 144, 1, 1, 1), (40, 7, 7, 576, 1, 1, 1), (300, 5, 3, 132, 1, 1, 1), (120, 1, 1, 4096, 1, 1, 1),
         (2, 113, 111, 36, 1, 1, 1), (9, 29, 31, 260, 2, 1, 1), (12, 15, 13, 1028, 2, 2, 2), (1, 1, 30000, 20, 1, 1, 1),
         (30000, 2, 1, 12, 1, 1, 1), (8, 33, 35, 64, 1, 0, 1), (2, 340, 340, 4, 1, 1, 1)]

WALK = [(10, 113, 111, 36, 1, 1, 1), (11, 112, 112, 32, 1, 1, 1), (30, 113, 111, 44, 2, 1, 1), (12, 60, 61, 100, 1, 2, 2),
        (1100, 1, 1, 4096, 1, 1, 1), (44000, 2, 1, 48, 1, 1, 1), (1, 1, 300000, 16, 1, 1, 1), (5300, 5, 3, 56, 1, 1, 1)]


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_against_the_oracle(case, signed, off):
    check(case, signed, off)


@pytest.mark.parametrize("signed, off", [(False, 0), (True, 1)])
@pytest.mark.parametrize("case", WALK, ids=lambda c: "x".join(map(str, c)))
def test_several_rounds_against_the_oracle(case, signed, off):
    n, h, w_, c, s, p, d = case
    with ax.AxLayer(ax._conv_desc((n, h, w_, c), (3, 3, c, 1), s, p, d, True), I.Quant(1.0, 0, 1.0, 0, None)) as layer:
        r, (_, oh, ow, _) = layer.route(), layer.out_shape()
    groups = c // 4
    step = r["workgroups"] * 1024 // groups * groups  # from one item of a thread to its next
    assert r["kernel"] == "depthwise" and n * oh * ow * groups > 4 * step
    check(case, signed, off)


def check(case, signed, off):
    n, h, w_, c, s, p, d = case
    rng = np.random.default_rng(c)
    lo, hi, dt = (-128, 128, np.int8) if signed else (0, 256, np.uint8)
    x = rng.integers(lo, hi, (n, h, w_, c)).astype(dt)
    w = rng.integers(lo, hi, (3, 3, c, 1)).astype(dt)
    lut = I.lut_signed_random(3) if signed else I.lut_random(3)
    q = I.Quant(0.02, -7, 0.01, 5, None) if signed else I.Quant(0.02, 7, 0.01, 120, None)
    acc_ref, y_ref = oracle.conv2d_ex(x, w, lut, s, p, q, dilation=d, depthwise=True, signed=signed)
    acc = torch.empty(acc_ref.size + off, dtype=torch.int32, device="cuda")
    y = torch.empty(acc_ref.size + off, dtype=torch.float32, device="cuda")
    assert acc_ref.size * 9 >= 4e6
    a, b = ax.ax_conv2d_ex(to_dev(x), to_dev(w), ax.lut_to_device(lut), s, p, q, dilation=d, depthwise=True,
                           acc_out=acc[off:], y_out=y[off:])
    torch.cuda.synchronize()
    assert_parity(a.cpu().numpy().reshape(acc_ref.shape), b.cpu().numpy().reshape(acc_ref.shape), acc_ref, y_ref)
