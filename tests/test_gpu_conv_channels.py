"""GPU parity of the forward and layer-gradient convolutions for channel counts that are no multiples of 64: pieces of 16
channels with a remainder, several taps in one step of 64, tiles of output channels with a remainder, stride classes with
and without taps.  Accumulators and float results bit-exact (one rounding of an exact integer)."""
import pytest

import oracle
import synth
from gpu_util import close, dev, host, qp_dev_from, require_gpu, same_ints
from test_gpu_products import _conv_operands

pytestmark = pytest.mark.gpu

SHAPES = [
    # N, C, H, W, K, R, S, stride, pad
    (40, 16, 32, 32, 16, 3, 3, 1, 1),     # four taps per step, the last step with three surplus pieces
    (9, 17, 33, 31, 47, 3, 3, 1, 1),      # 2 and 3 pieces per tap, one channel in the last; odd plane
    (6, 96, 27, 27, 200, 3, 3, 1, 1),     # 6 and 13 pieces, a last tile of 8 channels
    (5, 65, 15, 14, 129, 3, 3, 1, 1),     # one channel behind a tile of 64 / 128
    (300, 48, 5, 5, 63, 3, 3, 1, 1),      # tiny planes, 128-row tiles over many images
    (4, 64, 28, 28, 100, 3, 3, 1, 1),     # whole tiles on one side only
    (3, 200, 13, 17, 64, 1, 1, 1, 0),     # a single tap
    (8, 1, 65, 64, 33, 5, 5, 1, 2),       # one channel
    (4, 24, 40, 36, 40, 7, 7, 1, 3),      # 49 taps, pieces of two taps in a step
    (4, 24, 36, 36, 72, 3, 3, 2, 1),      # stride 2, even width: class pairs
    (4, 40, 35, 33, 72, 3, 3, 2, 1),      # ... odd sizes: classes of their own
    (6, 80, 30, 28, 48, 1, 1, 2, 0),      # ... three classes without taps, zeros written by the fourth
    (6, 80, 29, 28, 48, 1, 1, 2, 0),
    (3, 36, 40, 40, 50, 5, 4, 3, 2),      # stride 3, filter not square
    (2, 300, 14, 14, 260, 3, 3, 1, 1),    # 256-column tiles have to be declined or cut
    (200, 130, 12, 12, 250, 3, 3, 1, 1),  # many rows: 256x256 tiles with a remainder of 6 channels
    (3, 3, 40, 44, 192, 7, 7, 2, 3),      # few input channels: three blocks of 64 output channels on one band of rows
    (2, 5, 27, 24, 128, 5, 3, 1, 1),      # ... two, ragged band
    (3, 3, 64, 64, 64, 9, 9, 2, 4),       # more than 49 taps
    (2, 3, 96, 96, 64, 16, 16, 16, 0),    # patches
    (2, 20, 21, 21, 24, 3, 3, 5, 1),      # stride beyond 4: general kernel
]


@pytest.mark.parametrize("case", SHAPES)
def test_conv_channel_counts(case):
    q8t = require_gpu()
    g = synth.rng(sum(case))
    od, (sx, px), (sw, pw), (sg, pg), _ = _conv_operands(g, case)
    d = q8t.conv_desc(*case)
    dpx, dpw, dpg = (qp_dev_from(p) for p in (px, pw, pg))
    oy, oacc = oracle.qconv_fwd(od, sx, px, sw, pw)
    y, acc = q8t.qconv_fwd(d, dev(sx), dpx, dev(sw), dpw, want_acc=True)
    same_ints(host(acc), oacc)
    same_ints(host(y), oy)
    y, acc, stats = q8t.qconv_fwd_bn_stats(d, dev(sx), dpx, dev(sw), dpw, want_acc=True)
    same_ints(host(acc), oacc)
    yk = oy.astype("float64").transpose(1, 0, 2, 3).reshape(oy.shape[1], -1)
    close(host(stats)[0], yk.mean(axis=1))
    same_ints(host(stats)[1:], [yk.min(axis=1), yk.max(axis=1)])
    odx, oacc = oracle.qconv_dgrad(od, sg, pg, sw, pw)
    dx, acc = q8t.qconv_dgrad(d, dev(sg), dpg, dev(sw), dpw, want_acc=True)
    same_ints(host(acc), oacc)
    same_ints(host(dx), odx)


@pytest.mark.parametrize("case", [(7, 40, 19, 21, 72, 3, 3, 1, 1), (2, 3, 20, 24, 64, 3, 3, 1, 1)])
def test_conv_operand_at_any_address(case):
    # the relayout / the staged band of rows reads four codes at a time wherever the operand starts
    q8t = require_gpu()
    od, (sx, px), (sw, pw), _, _ = _conv_operands(synth.rng(3), case)
    _, oacc = oracle.qconv_fwd(od, sx, px, sw, pw)
    d = q8t.conv_desc(*case)
    for off in (1, 2, 3):
        flat = dev(sx.ravel())
        buf = flat.new_empty(flat.numel() + off)
        buf[off:] = flat
        _, acc = q8t.qconv_fwd(d, buf[off:].view(sx.shape), qp_dev_from(px), dev(sw), qp_dev_from(pw), want_acc=True)
        same_ints(host(acc), oacc)


@pytest.mark.parametrize("case", [
    (1024, 48, 1, 1, 80, 1, 1, 1, 0),     # planes of one position: several images per workgroup of the relayout, both ways
    (1030, 17, 2, 2, 33, 3, 3, 2, 1),     # ... the last workgroup short, odd numbers of bytes
    (1500, 16, 1, 3, 16, 3, 3, 1, 1),
    (1025, 97, 7, 9, 66, 1, 1, 1, 0),     # the most bytes of a plane that go this way, 63 positions
    (1026, 64, 8, 8, 24, 3, 3, 1, 1),     # 64 positions: one workgroup per plane again
    (1023, 48, 1, 2, 80, 1, 1, 1, 0),     # one image too few
    (2049, 320, 2, 2, 70, 2, 2, 1, 0),    # 4 positions on one side, 1 on the other
    (70001, 5, 1, 1, 130, 1, 1, 1, 0),    # many images per workgroup
])
def test_conv_tiny_planes(case):
    test_conv_channel_counts(case)


def test_conv_more_images_than_workgroups_of_a_launch():
    # 256 threads per image would be more than the 2^32 of a launch
    q8t = require_gpu()
    case = ((1 << 24) + 5, 4, 1, 1, 1, 1, 1, 1, 0)
    od, (sx, px), (sw, pw), _, _ = _conv_operands(synth.rng(5), case)
    _, oacc = oracle.qconv_fwd(od, sx, px, sw, pw)
    _, acc = q8t.qconv_fwd(q8t.conv_desc(*case), dev(sx), qp_dev_from(px), dev(sw), qp_dev_from(pw), want_acc=True)
    same_ints(host(acc), oacc)


@pytest.mark.parametrize("case", [
    (2, 3, 41, 45, 64, 7, 7, 2, 3),       # row ends with 1, 2 and 3 codes in the last dword, odd planes
    (16, 1, 30, 58, 128, 5, 5, 1, 2),
    (16, 4, 19, 27, 64, 3, 3, 1, 1),
    (128, 3, 9, 259, 128, 7, 8, 2, 3),    # rows of more than 64 dwords, the last one ragged
    (4, 2, 7, 2, 64, 3, 3, 1, 1),         # a single, ragged dword
    (2, 2, 30, 3, 64, 7, 7, 1, 3),
])
def test_conv_few_channels_ragged_rows(case):
    test_conv_channel_counts(case)


@pytest.mark.parametrize("case", [
    (6, 80, 30, 28, 200, 1, 1, 2, 0),     # channel-contiguous layer gradient, three classes without taps
    (6, 80, 29, 28, 200, 1, 1, 2, 0),
    (3, 200, 13, 17, 300, 1, 1, 1, 0),    # ... a single tap, both ways
    (8, 24, 40, 36, 40, 7, 7, 1, 3),      # ... 49 taps
    (4, 300, 14, 14, 260, 3, 3, 1, 1),
    (5, 472, 7, 4, 1, 7, 7, 1, 3),        # few results, long reduction: general kernel, split
    (2, 5, 27, 24, 128, 5, 3, 1, 1),      # general product, first-layer kernel with statistics
    (4, 1, 11, 18, 80, 1, 1, 1, 0),       # general product, statistics in a pass of their own
    (16, 8, 12, 12, 64, 5, 5, 1, 2),      # im2col rows, one tile width; surplus columns 200 .. 255
    (16, 20, 12, 12, 512, 7, 7, 2, 3),    # ... 128-wide tiles, statistics in a pass of their own
    (57, 5, 8, 5, 64, 7, 7, 2, 3),        # ... rows that are no whole dwords, last row tile short
    (2, 8, 4, 4, 64, 7, 7, 1, 3),         # ... fewer positions than a tile, most taps in the padding
])
def test_conv_forms(case):
    test_conv_channel_counts(case)


def test_conv_im2col_rows_at_odd_addresses():
    import torch
    q8t = require_gpu()
    case = (16, 8, 12, 12, 64, 5, 5, 1, 2)    # whole dwords in a row, but not at the operand's address
    od, (sx, px), (sw, pw), _, _ = _conv_operands(synth.rng(208), case)
    _, oacc = oracle.qconv_fwd(od, sx, px, sw, pw)
    x = dev(sx)
    for off in (1, 2, 3):
        buf = torch.empty(x.numel() + off, dtype=torch.int8, device=x.device)
        shifted = buf[off:].view(x.shape)
        shifted.copy_(x)
        _, acc = q8t.qconv_fwd(q8t.conv_desc(*case), shifted, qp_dev_from(px), dev(sw), qp_dev_from(pw), want_acc=True)
        same_ints(host(acc), oacc)
