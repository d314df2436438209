"""Layers of few output pixels (whole table in LDS, taps over the lanes) and tiny layers (several
threads per output) against the oracle, at the edges of their tiles: pixels per tile 1, 2, 4, 7, 8,
channel groups and tap slices that do not divide, workgroups that walk over several tiles, the longest
sums, byte-granular operands, unaligned pointers.  Every case asserts which kernel it runs."""

import numpy as np
import pytest
import torch

from gpu_common import assert_parity, check_layer, to_dev
from oracle import oracle
from paper_2002_09481_amd import binding as ax
from paper_2002_09481_amd import inputs as I

pytestmark = pytest.mark.gpu

L = I.Layer


def _dense(M, K, N):
    return L("dense", M, 1, 1, K, 1, 1, N, dense=True, x_dist="relu", w_dist="normal")


def _conv(N, H, W, Cin, k, Cout, stride=1, pad=0):
    return L("conv", N, H, W, Cin, k, k, Cout, stride, pad, x_dist="relu", w_dist="normal")


FEW = [_dense(1, 2048, 1000), _dense(2, 2051, 1001), _dense(3, 4100, 340), _dense(7, 1536, 257), _dense(8, 1024, 516),
       _dense(9, 777, 333), _dense(33, 2048, 1000), _dense(50, 516, 1030), _dense(64, 100, 1000), _dense(1, 32768, 132),
       _conv(1, 7, 7, 512, 3, 128, 1, 1), _conv(1, 14, 14, 256, 1, 516), _conv(1, 13, 15, 260, 1, 300, 2),
       _conv(2, 9, 5, 132, 3, 70, 2, 1), _conv(1, 14, 13, 50, 5, 70, 1, 2), _conv(1, 28, 28, 128, 1, 512),
       _conv(3, 6, 7, 64, 3, 257, 1, 2)]
# more than twice as many tiles as compute units, so that a workgroup walks over three, with ragged last
# tiles of pixels and channels: dwords, then the byte form
WALK = [_conv(3, 7, 7, 2048, 1, 512), _dense(201, 208, 1494), _dense(332, 112, 1926), _dense(5634, 1000, 5),
        _dense(5692, 80, 47), _dense(105, 3684, 291), _dense(129, 95, 2681), _dense(78, 399, 915), _dense(587, 3999, 19)]
TINY = [_conv(1, 16, 16, 8, 3, 8, 1, 1), _conv(1, 3, 3, 4, 3, 5, 1, 1), _dense(1, 1, 1), _dense(1, 2048, 100), _dense(2, 63, 7), _dense(1, 32768, 68),
        _dense(1, 64, 1001), _dense(1, 32768, 3), _conv(2, 20, 20, 3, 5, 9, 2, 2), _conv(1, 60, 60, 4, 1, 70)]


def _at(t, off):
    """A copy of a device tensor that starts `off` elements past an allocation's start."""
    flat = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
    v = flat[off:off + t.numel()]
    v.copy_(t.reshape(-1))
    return v.view(t.shape)


def _desc(layer):
    if layer.dense:
        return ax._dense_desc(layer.N, layer.K, layer.Cout)
    return ax._conv_desc((layer.N, layer.H, layer.W, layer.Cin), (layer.KH, layer.KW, layer.Cin, layer.Cout), layer.stride, layer.pad)


def _route(layer):
    with ax.AxLayer(_desc(layer), I.Quant(1.0, 0, 1.0, 0, None)) as h:
        assert h.plan()["variant"] == 1 and h.prepared_bytes == 0
        return h.route()


@pytest.mark.parametrize("layer", FEW + WALK + TINY, ids=lambda l: "%dx%dx%d" % (l.M, l.K, l.Cout))
def test_against_the_oracle(layer):
    r = _route(layer)
    assert r["kernel"] == ("direct" if layer in TINY else "fewpix")
    if layer in WALK:
        assert r["tiles"] > 2 * r["workgroups"]
    check_layer(layer, 3, I.lut_random_error(5))


@pytest.mark.parametrize("layer", [WALK[1], WALK[7]], ids=["dwords", "bytes"])
def test_walk_with_signed_codes(layer):
    rng = np.random.default_rng(13)
    x = rng.integers(-128, 128, (layer.M, 1, 1, layer.K), dtype=np.int8)
    w = rng.integers(-128, 128, (1, 1, layer.K, layer.Cout), dtype=np.int8)
    lut = I.lut_signed_random_error(4)
    q = I.Quant(0.02, -7, 0.01, 5, None)
    acc, y = ax.ax_conv2d_ex(to_dev(x), to_dev(w), ax.lut_to_device(lut), 1, 0, q)
    torch.cuda.synchronize()
    assert_parity(acc.cpu().numpy(), y.cpu().numpy(), *oracle.conv2d_ex(x, w, lut, 1, 0, q, signed=True))


@pytest.mark.parametrize("entry", [65535, 32767, -32768])
def test_longest_sums_of_the_largest_entries(entry):
    """32768 taps of one entry: the sums of the unsigned form end just under 2^31, those of the signed form
    at the entry's own sign; neighbouring sums share 64-bit additions."""
    M, K, N = 2, 32768, 597
    assert _route(_dense(M, K, N))["kernel"] == "fewpix"
    dt = torch.uint8 if entry == 65535 else torch.int8
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.randint(0, 128, (M, 1, 1, K), generator=g, device="cuda", dtype=torch.uint8).view(dt)
    w = torch.randint(0, 128, (1, 1, K, N), generator=g, device="cuda", dtype=torch.uint8).view(dt)
    lut = torch.full((65536,), -1 if entry == 65535 else entry, dtype=torch.int16, device="cuda")
    acc, _ = ax.ax_conv2d_ex(x, w, lut, 1, 0, I.Quant(1.0, 0, 1.0, 0, None))
    assert torch.equal(acc, torch.full_like(acc, K * entry))


@pytest.mark.parametrize("seed", range(40))
def test_random_layers_of_the_automatic_choice(seed):
    """No overrides: shapes drawn around the lines between the direct, the few-pixel and the table-tile
    kernels, both code types, operands at any byte and tables at any entry."""
    rng = np.random.default_rng(9100 + seed)
    lg = lambda lo, hi: int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))
    while True:
        k, s, d = int(rng.choice([1, 1, 3, 5])), int(rng.choice([1, 1, 2])), int(rng.choice([1, 1, 2]))
        n, hh, ww, cin, cout = int(rng.choice([1, 1, 2, 3])), lg(1, 40), lg(1, 40), lg(3, 1024), lg(4, 1200)
        pad = int(rng.integers(0, d * (k // 2) + 1))
        if min(hh, ww) + 2 * pad <= d * (k - 1) or k * k * cin > 32768:
            continue
        oh, ow = (hh + 2 * pad - d * (k - 1) - 1) // s + 1, (ww + 2 * pad - d * (k - 1) - 1) // s + 1
        if 2e5 <= n * oh * ow * k * k * cin * cout <= 6e7:
            break
    signed = bool(rng.random() < 0.4)
    lo, hi, dt = (-128, 128, np.int8) if signed else (0, 256, np.uint8)
    x = rng.integers(lo, hi, (n, hh, ww, cin)).astype(dt)
    w = rng.integers(lo, hi, (k, k, cin, cout)).astype(dt)
    lut = I.lut_signed_random_error(seed) if signed else I.lut_random_error(seed)
    q = I.Quant(0.02, -7, 0.01, 5, None) if signed else I.Quant(0.02, 7, 0.01, 120, None)
    off = [int(v) for v in rng.integers(0, 4, 3)]
    ld = _at(ax.lut_to_device(lut).view(torch.int16).reshape(-1), off[2])
    acc, y = ax.ax_conv2d_ex(_at(to_dev(x), off[0]), _at(to_dev(w), off[1]), ld, s, pad, q, d)
    torch.cuda.synchronize()
    assert_parity(acc.cpu().numpy(), y.cpu().numpy(), *oracle.conv2d_ex(x, w, lut, s, pad, q, dilation=d, signed=signed))


@pytest.mark.parametrize("shape", [(1, 7, 7, 256, 3, 128, 1, 1, 2), (2, 13, 9, 66, 3, 65, 2, 2, 1), (1, 5, 5, 8, 3, 9, 1, 1, 1)],
                         ids=["dwords", "bytes", "tiny"])
def test_signed_codes_pad_code_and_dilation(shape):
    n, hh, ww, cin, k, cout, stride, pad, dil = shape
    rng = np.random.default_rng(11)
    x = rng.integers(-128, 128, (n, hh, ww, cin), dtype=np.int8)
    w = rng.integers(-128, 128, (k, k, cin, cout), dtype=np.int8)
    lut = I.lut_signed_random_error(3)
    q = I.Quant(0.02, -7, 0.01, 5, -100)
    acc, y = ax.ax_conv2d_ex(to_dev(x), to_dev(w), ax.lut_to_device(lut), stride, pad, q, dil)
    torch.cuda.synchronize()
    acc_ref, y_ref = oracle.conv2d_ex(x, w, lut, stride, pad, q, dilation=dil, signed=True)
    assert_parity(acc.cpu().numpy(), y.cpu().numpy(), acc_ref, y_ref)


@pytest.mark.parametrize("off", [(1, 0, 0), (0, 1, 0), (0, 0, 1), (2, 3, 1)])
def test_unaligned_operands(off):
    """Operands that start at any byte, tables at any entry."""
    layer = _dense(5, 1024, 516)
    x, w, q = I.make_operands(layer, 4)
    lut = I.lut_random_error(6)

    xd = _at(to_dev(x.reshape(5, -1)), off[0])
    wd = _at(to_dev(w.reshape(1024, 516)), off[1])
    ld = _at(ax.lut_to_device(lut).view(torch.int16).reshape(-1), off[2])
    acc, y = ax.ax_dense(xd, wd, ld, q)
    torch.cuda.synchronize()
    acc_ref, y_ref = oracle.dense(x.reshape(5, -1), w.reshape(1024, 516), lut, q)
    assert_parity(acc.cpu().numpy(), y.cpu().numpy(), acc_ref, y_ref)


def _us(call):
    """Microseconds of a call among others (the smallest of eight means of 20)."""
    best = 1e9
    for _ in range(8):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(20):
            call()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 50.0)
    return best


@pytest.mark.parametrize("which", ["x", "w", "lut"])
def test_unaligned_operands_cost_no_other_form(which):
    """A layer chosen for the few-pixel kernel stays as fast whatever byte its operands start at (the choice
    knows the geometry only): its results are the oracle's, and a call takes at most 1.35 times the aligned
    one's time.  Loads that straddle a cache line cost a few percent; a byte-by-byte form took 1.7 times."""
    layer = _conv(1, 14, 14, 256, 3, 256, 1, 1)
    x, w, q = I.make_operands(layer, 8)
    lut = I.lut_random_error(9)
    xd, wd, ld = to_dev(x), to_dev(w), ax.lut_to_device(lut).view(torch.int16).reshape(-1)
    moved = {"x": (_at(xd, 1), wd, ld), "w": (xd, _at(wd, 3), ld), "lut": (xd, wd, _at(ld, 1))}[which]
    acc = torch.empty((1, 14, 14, 256), dtype=torch.int32, device="cuda")
    y = torch.empty(acc.shape, dtype=torch.float32, device="cuda")

    def us(a, b, t):
        return _us(lambda: ax.ax_conv2d(a, b, t, 1, 1, q, acc_out=acc, y_out=y))

    aligned, unaligned = us(xd, wd, ld), us(*moved)
    assert_parity(acc.cpu().numpy(), y.cpu().numpy(), *oracle.conv2d(x, w, lut, 1, 1, q))
    assert unaligned < 1.35 * aligned, (aligned, unaligned)


@pytest.mark.parametrize("M, K, N", [(8, 8192, 1001), (1, 32768, 497), (48, 13600, 39), (9, 3096, 709)])
def test_odd_channel_counts_cost_no_other_form(M, K, N):
    """A channel count that is no multiple of four costs what the next multiple costs: filters are read by the
    dword either way (byte by byte the first two took 1.5 and 2.1 times as long)."""
    layer = _dense(M, K, N)
    x, w, q = I.make_operands(layer, 10)
    lut = I.lut_random_error(11)
    xd, ld = to_dev(x).view(M, K), ax.lut_to_device(lut)
    wide = -(-N // 4) * 4
    wd = to_dev(w).view(K, N)
    w4 = torch.zeros((K, wide), dtype=torch.uint8, device="cuda")
    w4[:, :N] = wd

    def prepared(wt, n):
        h = ax.AxLayer(ax._dense_desc(M, K, n), q)
        assert h.plan()["variant"] == 1
        h.prepare(wt, ld)
        acc, y = h.run(xd)
        return h, acc, y

    h, acc, y = prepared(wd, N)
    h4, acc4, y4 = prepared(w4, wide)
    odd, even = _us(lambda: h.run(xd, acc, y)), _us(lambda: h4.run(xd, acc4, y4))
    acc_ref, y_ref = oracle.dense(x.reshape(M, K), w.reshape(K, N), lut, q)
    assert_parity(acc.cpu().numpy(), y.cpu().numpy(), acc_ref, y_ref)
    assert odd < 1.25 * even, (odd, even)
