"""Table tiles and what prepares their activations, at the sizes where each form begins and ends: heights of
a tile, odd and even chunk counts, activations read in place and from their copy, patch stripes of
whole and partial rows, pieces of shared tiles.  Against the oracle: int32 accumulators bit exact."""

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2002_09481_amd import binding as ax
from paper_2002_09481_amd import inputs as I

import gpu_common as G
from test_gpu_variants import _operands

pytestmark = pytest.mark.gpu

TUNE = dict(variant=2, split_k=0, tile=0, row_tiles=0, share_order=0, combine=0, tables=0)


def _run(shape, stride, pad, dilation, signed, tune, small_workspace=False, offset=0):
    x, w, q = _operands(shape, sum(shape) + 2 * signed, signed)
    lut = I.lut_signed_random_error(7) if signed else I.lut_random_error(7)
    want, y_want = oracle.conv2d_ex(x, w, lut, stride, pad, q, dilation=dilation, signed=signed)
    with ax.AxLayer(ax._conv_desc(x.shape, w.shape, stride, pad, dilation, signed=signed), q,
                    tune=dict(TUNE, **tune)) as h:
        assert h.plan()["variant"] == tune.get("variant", 2)
        h.prepare(G.to_dev(w), ax.lut_to_device(lut))
        buf = torch.empty(x.size + offset, dtype=torch.int8 if signed else torch.uint8, device="cuda")
        xd = buf[offset:].view(x.shape)
        xd.copy_(G.to_dev(x))
        ws = torch.empty(256, dtype=torch.uint8, device="cuda") if small_workspace else None
        for call in range(2):
            acc, y = h.run(xd, workspace=ws)
            torch.cuda.synchronize()
            G.assert_parity(acc.cpu().numpy(), y.cpu().numpy(), want, y_want, "%s %s call %d" % (shape, tune, call))
        return h.plan()


# one tile of every height class: 64 lane elements, the last with double-buffered rows (2048), the first
# without (2049), the tallest (4096) and one more; one, two and three chunks, five with a ragged last one
@pytest.mark.parametrize("tables", [1, 2])
@pytest.mark.parametrize("K", [16, 32, 48, 70])
@pytest.mark.parametrize("M", [1, 64, 65, 2048, 2049, 4096, 4097])
def test_tile_heights_and_chunk_counts(M, K, tables):
    _run((M, 1, 1, K, 1, 1, 9), 1, 0, 1, False, dict(row_tiles=1 if M <= 4096 else 2, split_k=1, tables=tables))


# (shape, stride, pad, dilation): copies with border, by output pixel, with other strides and dilations; rows of
# more than 32767 pixels with padding
VIEWS = [
    ((2, 9, 11, 16, 3, 3, 9), 1, 1, 1), ((2, 9, 11, 32, 3, 3, 8), 2, 1, 1), ((1, 12, 10, 48, 3, 3, 17), 1, 2, 2),
    ((3, 7, 9, 144, 1, 1, 8), 2, 0, 1), ((2, 6, 5, 64, 1, 1, 70), 1, 0, 1), ((1, 8, 8, 16, 5, 3, 8), 1, (4, 0), 1),
    ((1, 2, 32800, 16, 1, 3, 5), 1, (0, 1), 1),
]


@pytest.mark.parametrize("copied", [True, False])
@pytest.mark.parametrize("case", VIEWS, ids=lambda c: "x".join(map(str, c[0])))
def test_a_workspace_with_room_for_the_copy_receives_it(case, copied):
    """Without shared tiles the copy of the activations is all that a call keeps in its workspace: a buffer of just
    its size is written from end to end, one that is a byte short of the copy without border is left alone and the
    activations are read in place."""
    (N, H, W, C, KH, KW, _), stride, pad, dilation = case
    ph, pw = ax._pair(pad)
    x, w, q = _operands(case[0], sum(case[0]), False)
    lut = I.lut_random_error(7)
    with ax.AxLayer(ax._conv_desc(x.shape, w.shape, stride, pad, dilation), q, tune=dict(TUNE, split_k=1)) as h:
        plain = h.out_shape()[1] * h.out_shape()[2] if KH == KW == 1 and not pad else H * W
        border = (H + 2 * ph) * (W + 2 * pw) if pad else plain
        if N * border * C > h.workspace_bytes:  # no room for the border in any workspace that the layer asks for
            border = plain
        copied = copied and (C > 16 or border != H * W)
        h.prepare(G.to_dev(w), ax.lut_to_device(lut))
        buf = torch.empty(N * (border if copied else plain) * C - (0 if copied else 1), dtype=torch.uint8, device="cuda")
        want = oracle.conv2d_ex(x, w, lut, stride, pad, q, dilation=dilation)
        for fill in (0xA5, 0x5A):  # a byte that is the filler in one run is another in the next
            buf.fill_(fill)
            acc, y = h.run(G.to_dev(x), workspace=buf)
            torch.cuda.synchronize()
            G.assert_parity(acc.cpu().numpy(), y.cpu().numpy(), *want)
            kept = buf == fill
            assert bool(kept.all()) == (not copied)
            left = kept if fill == 0xA5 else left & kept
        assert not copied or not bool(left.any())


@pytest.mark.parametrize("signed, small_workspace", [(False, False), (False, True), (True, False)])  # signed codes need their copy
@pytest.mark.parametrize("case", VIEWS, ids=lambda c: "x".join(map(str, c[0])))
def test_activations_in_place_and_from_their_copy(case, signed, small_workspace):
    _run(*case, signed, dict(split_k=1), small_workspace)


# channel counts or base addresses that rule out aligned 16-byte reads: stripes of one pixel, of a ragged last
# column and row, of several rows, wholly in the padding; strides beyond the filter, wide dilations; the images
# as one row; too wide for the stage
PATCHES = [
    ((1, 1, 1, 1, 1, 1, 5), 1, 0, 1), ((3, 17, 1, 3, 3, 1, 8), 1, (1, 0), 1), ((1, 5, 300, 3, 3, 3, 8), 1, 1, 1),
    ((70, 19, 23, 3, 3, 3, 4), 1, 1, 1), ((300, 9, 6, 1, 2, 2, 4), 1, 0, 1), ((2, 21, 26, 5, 3, 3, 8), 5, 1, 1),
    ((1, 6, 6, 4, 1, 1, 8), 1, 7, 1), ((2, 30, 28, 7, 3, 3, 8), 1, 9, 9), ((40, 1, 1, 100, 1, 1, 8), 1, 0, 1),
    ((5, 8, 6, 21, 1, 1, 8), 1, 0, 1), ((5, 9, 7, 21, 1, 1, 8), 2, 0, 1), ((2, 5, 40, 1030, 3, 3, 8), 1, 1, 1),
    ((2, 3, 3, 4097, 1, 1, 8), 1, 0, 1),
    # only the rows that taps read: one output row a block, several with a ragged last one, a stride beyond the filter, one filter row
    ((1, 40, 50, 3, 3, 3, 8), 1, 12, 12), ((130, 21, 12, 3, 3, 3, 4), 1, 8, 8), ((200, 41, 6, 5, 2, 2, 4), (6, 1), 1, 1), ((300, 26, 9, 3, 1, 3, 4), (5, 1), 0, 1),
]


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("case", PATCHES, ids=lambda c: "x".join(map(str, c[0])))
def test_patches_copied_out(case, signed):
    _run(*case, signed, {})


def test_activations_at_any_byte():
    for offset in (1, 4, 8):
        _run((2, 9, 11, 32, 3, 3, 9), 1, 1, 1, False, {}, offset=offset)


@pytest.mark.parametrize("combine", [1, 2])
@pytest.mark.parametrize("split", [2, 3, 7])
@pytest.mark.parametrize("case", [((3, 5, 5, 64, 3, 3, 20), 1, 1, 1), ((1, 48, 48, 64, 3, 3, 9), 1, 1, 1), ((130, 1, 1, 500, 1, 1, 30), 1, 0, 1)],
                         ids=lambda c: "x".join(map(str, c[0])))
def test_pieces_of_shared_tiles(case, split, combine):
    plan = _run(*case, False, dict(split_k=split, combine=combine))
    assert plan["pieces"] > 0 and plan["combine"] == combine


def test_channel_lanes_and_a_sum_of_more_taps_than_sixteen_bits_hold():
    _run((60, 1, 1, 200, 1, 1, 70), 1, 0, 1, False, dict(variant=3))
    for variant in (2, 3):
        _run((3, 1, 1, 32768, 1, 1, 9), 1, 0, 1, False, dict(variant=variant))


@pytest.mark.parametrize("split, combine", [(1, 0), (3, 1), (3, 2)])
@pytest.mark.parametrize("variant", [2, 3])
@pytest.mark.parametrize("entry", [65535, 0, 32767, -32768])
def test_longest_sums_of_the_largest_entries(entry, variant, split, combine):
    """32768 taps of one entry: byte sums, their corrections and the 64-bit dequantization at their limits (the unsigned
    sum ends just under 2^31), whole and in pieces."""
    signed = entry in (32767, -32768)
    x, w, q = _operands((3, 1, 1, 32768, 1, 1, 9), 5 + signed, signed)
    q = I.Quant(q.x_scale, 127 if signed else 255, q.w_scale, -128 if signed else 255, None)
    lut = np.full(65536, entry, np.int16 if signed else np.uint16)
    with ax.AxLayer(ax._conv_desc(x.shape, w.shape, 1, 0, signed=signed), q,
                    tune=dict(TUNE, variant=variant, split_k=split, combine=combine)) as h:
        assert (h.plan()["pieces"] > 0) == (split > 1)
        h.prepare(G.to_dev(w), ax.lut_to_device(lut))
        acc, y = h.run(G.to_dev(x))
        torch.cuda.synchronize()
    want, y_want = oracle.conv2d_ex(x, w, lut, 1, 0, q, signed=signed)
    assert bool((want == 32768 * entry).all())
    G.assert_parity(acc.cpu().numpy(), y.cpu().numpy(), want, y_want)


def test_stripes_against_the_general_patch_copy():
    """The staged copy and the general one (sums of more than 4096 taps) give the same patches: a layer, and the same
    layer with zero channels appended until only the general form takes it, differ by the table's value at
    code 0 alone."""
    rng = np.random.default_rng(3)
    x = rng.integers(0, 256, (2, 7, 9, 5), dtype=np.uint8)
    w = rng.integers(0, 256, (3, 3, 5, 6), dtype=np.uint8)
    lut = I.lut_random_error(11).copy().reshape(256, 256)
    lut[0, 0] = 0
    q = I.Quant(0.02, 0, 0.01, 0, None)
    wide_x, wide_w = np.zeros((2, 7, 9, 501), np.uint8), np.zeros((3, 3, 501, 6), np.uint8)
    wide_x[..., :5], wide_w[:, :, :5] = x, w
    out = []
    for a, b in ((x, w), (wide_x, wide_w)):
        with ax.AxLayer(ax._conv_desc(a.shape, b.shape, 1, 1), q, tune=TUNE) as h:
            h.prepare(G.to_dev(b), ax.lut_to_device(lut))
            out.append(h.run(G.to_dev(a))[0].cpu().numpy())
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("offset", [1, 16, 128, 0])
def test_a_workspace_off_its_alignment_stays_unused(offset):
    """A layer that reads its activations in place and has no shared tiles needs no scratch: a buffer that is not
    256-byte aligned is accepted and not written, an aligned one of the full size receives the copy."""
    x, w, q = _operands((2, 9, 11, 32, 3, 3, 9), 60, False)
    lut = I.lut_random_error(7)
    with ax.AxLayer(ax._conv_desc(x.shape, w.shape, 1, 1), q, tune=dict(TUNE, split_k=1)) as h:
        assert h.plan()["pieces"] == 0
        h.prepare(G.to_dev(w), ax.lut_to_device(lut))
        buf = torch.full((h.workspace_bytes + 512,), 0xA5, dtype=torch.uint8, device="cuda")
        start = -buf.data_ptr() % 256
        acc, y = h.run(G.to_dev(x), workspace=buf[start + offset:start + offset + h.workspace_bytes])
        torch.cuda.synchronize()
        G.assert_parity(acc.cpu().numpy(), y.cpu().numpy(), *oracle.conv2d_ex(x, w, lut, 1, 1, q))
        assert bool((buf == 0xA5).all()) == (offset != 0)


def test_more_images_than_a_launch_holds_blocks():
    """A block per image would be a launch of 2^32 threads."""
    N = 1 << 24
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x = torch.randint(0, 256, (N, 2, 2, 1), generator=g, device="cuda", dtype=torch.uint8)
    w = np.array([3, 200, 0, 255, 17, 90, 128, 64], np.uint8).reshape(2, 2, 1, 2)
    lut = I.lut_random_error(2)
    with ax.AxLayer(ax._conv_desc(x.shape, w.shape, 1, 0), I.Quant(1.0, 0, 1.0, 0, None), tune=TUNE) as h:
        h.prepare(G.to_dev(w), ax.lut_to_device(lut))
        acc, _ = h.run(x, y_out=False)
    table = torch.from_numpy(lut.astype(np.int32).reshape(256, 256)).cuda()
    want = sum(table[x.view(N, 4)[:, t].long()][:, torch.from_numpy(w.reshape(4, 2)[t].astype(np.int64)).cuda()] for t in range(4))
    assert torch.equal(acc.view(N, 2), want)


@pytest.mark.parametrize("split", [1, 2])
@pytest.mark.parametrize("offset", [0, 1, 2, 4])
@pytest.mark.parametrize("channels", [1, 2, 4, 6, 12, 20, 23])
def test_output_pieces_of_every_alignment(channels, offset, split):
    """Outputs in pieces of 16, 8 and 4 bytes, by channel count and start of the tensors; last columns and rows of a tile."""
    x, w, q = _operands((5, 7, 9, 16, 3, 3, channels), channels, False)
    lut = I.lut_random_error(7)
    want = oracle.conv2d_ex(x, w, lut, 1, 1, q)
    with ax.AxLayer(ax._conv_desc(x.shape, w.shape, 1, 1), q, tune=dict(TUNE, split_k=split, combine=2)) as h:
        h.prepare(G.to_dev(w), ax.lut_to_device(lut))
        n = 5 * 7 * 9 * channels
        bufs = [torch.full((n + 16,), 77, dtype=t, device="cuda") for t in (torch.int32, torch.float32)]
        views = [b[offset:offset + n].view(h.out_shape()) for b in bufs]
        acc, y = h.run(G.to_dev(x), *views)
        torch.cuda.synchronize()
        G.assert_parity(acc.cpu().numpy(), y.cpu().numpy(), *want)
        for b in bufs:
            assert bool((b[:offset] == 77).all()) and bool((b[offset + n:] == 77).all())


def test_pieces_of_more_tiles_than_one_row_of_a_launch():
    """The second kernel takes 64 lane elements per block: 16 tables of 67 million pixels are 2^24 blocks and some."""
    M, K, T = (1 << 26) + 64, 17, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    x = torch.randint(0, 256, (M, K), generator=g, device="cuda", dtype=torch.uint8)
    w = torch.randint(0, 256, (K, 1), generator=g, device="cuda", dtype=torch.uint8)
    luts = torch.randint(-32768, 32768, (T, 65536), generator=g, device="cuda", dtype=torch.int16)
    with ax.AxLayer(ax._dense_desc(M, K, 1), I.Quant(1.0, 0, 1.0, 0, None), T, tune=dict(TUNE, split_k=1, combine=1)) as h:
        assert h.plan()["pieces"] > 0 and h.plan()["combine"] == 1
        h.prepare(w, luts)
        acc = h.run(x, y_out=False)[0].view(T, M)
    for t in (0, 7, 15):
        table = (luts[t].to(torch.int32) & 0xFFFF).view(256, 256)
        for part in (slice(0, 1 << 20), slice(M // 2, M // 2 + (1 << 20)), slice(M - (1 << 20), M)):
            want = sum(table[:, int(w[k, 0])][x[part, k].long()] for k in range(K))
            assert torch.equal(acc[t, part], want)


# filters turned for channel lanes: columns past the last whole four, one column, more than a block's 1024; rows of
# less than a chunk and with a ragged last one; filters that start off a dword boundary
@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("K,Cout", [(3, 1), (16, 3), (17, 70), (147, 4), (33, 1027), (64, 2048)])
def test_channel_lanes_turn_filters_of_any_width_and_alignment(K, Cout, offset, signed):
    x, w, q = _operands((5, 1, 1, K, 1, 1, Cout), K + Cout, signed)
    lut = I.lut_signed_random_error(7) if signed else I.lut_random_error(7)
    want, y_want = oracle.conv2d_ex(x, w, lut, 1, 0, q, signed=signed)
    with ax.AxLayer(ax._conv_desc(x.shape, w.shape, 1, 0, signed=signed), q, tune=dict(TUNE, variant=3)) as h:
        assert h.plan()["variant"] == 3
        buf = torch.empty(w.size + offset, dtype=torch.int8 if signed else torch.uint8, device="cuda")
        wd = buf[offset:].view(w.shape)
        wd.copy_(G.to_dev(w))
        h.prepare(wd, ax.lut_to_device(lut))
        acc, y = h.run(G.to_dev(x))
        torch.cuda.synchronize()
        G.assert_parity(acc.cpu().numpy(), y.cpu().numpy(), want, y_want, "K %d Cout %d offset %d" % (K, Cout, offset))


# pieces combined by the workgroup that ends last: one group of 64 elements per wave, one wave with two, half and full
# height with ragged last groups; an even and an odd number of pieces
@pytest.mark.parametrize("tables", [1, 2])
@pytest.mark.parametrize("split_k", [2, 3, 5])
@pytest.mark.parametrize("M", [40, 512, 513, 2000, 2049, 4033])
def test_pieces_combined_in_the_kernel(M, split_k, tables):
    plan = _run((M, 1, 1, 96, 1, 1, 9), 1, 0, 1, False, dict(row_tiles=1, split_k=split_k, combine=2, tables=tables))
    assert plan["pieces"] > 0 and plan["combine"] == 2


# as above, every remainder of four pieces (a single group's step) and of two (a pair of groups'): 1, 2, 3 and 8 groups per wave
@pytest.mark.parametrize("split_k", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("M", [64, 1024, 1100, 4096])
def test_every_number_of_pieces_combined_in_the_kernel(M, split_k):
    plan = _run((M, 1, 1, 128, 1, 1, 9), 1, 0, 1, False, dict(row_tiles=1, split_k=split_k, combine=2, tables=1))
    assert plan["pieces"] == 2 * split_k and plan["combine"] == 2


# activations read in place above half the height, whole tiles and pieces (summed by the workgroup that ends last and by a
# second launch): odd and even chunk counts, one chunk more than pieces
@pytest.mark.parametrize("tables", [1, 2])
@pytest.mark.parametrize("split_k, combine", [(1, 0), (2, 1), (4, 2), (8, 2)])
@pytest.mark.parametrize("C, KH, KW", [(16, 3, 3), (32, 3, 3), (16, 1, 2)])
def test_tall_tiles_read_in_place(C, KH, KW, split_k, combine, tables):
    x, w, q = _operands((1, 50, 52, C, KH, KW, 9), C + split_k, False)
    lut = I.lut_random_error(7)
    want, y_want = oracle.conv2d_ex(x, w, lut, 1, 1, q)
    with ax.AxLayer(ax._conv_desc(x.shape, w.shape, 1, 1), q,
                    tune=dict(TUNE, row_tiles=1, split_k=split_k, combine=combine, tables=tables)) as h:
        _, OH, OW, _ = h.out_shape()
        height = -(-OH * OW // 64) * 64
        assert 2048 < height <= 4096
        pieces = 2 * h.plan()["workgroups"] * height * 36 if h.plan()["pieces"] else 256  # and no room for a copy
        h.prepare(G.to_dev(w), ax.lut_to_device(lut))
        acc, y = h.run(G.to_dev(x), workspace=torch.empty(pieces, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        G.assert_parity(acc.cpu().numpy(), y.cpu().numpy(), want, y_want, "%dx%dx%d %d" % (C, KH, KW, split_k))
