"""GPU parity of the general convolution where its pieces are copied to LDS: reductions that end in the first or the second half
of a step, one step and several, taps that begin inside a step, padded taps with a last piece of few channels, 128x128 tiles
(256 of them and more) beside 128x64 ones, class pairs.  Accumulators and float results bit-exact."""
import pytest

import oracle
import synth
from gpu_util import dev, host, qp_dev_from, require_gpu, same_ints
from test_gpu_products import _conv_operands

pytestmark = pytest.mark.gpu

SHAPES = [
    # N, C, H, W, K, R, S, stride, pad
    (8, 16, 12, 12, 64, 2, 2, 1, 1),       # one half of a step
    (8, 32, 12, 12, 64, 2, 2, 1, 1),       # a whole step
    (8, 48, 12, 12, 80, 2, 2, 1, 1),       # a step and a half; taps of three pieces
    (8, 33, 11, 13, 70, 3, 3, 1, 2),       # one channel in the last piece, two rows of padding
    (4, 31, 9, 9, 129, 5, 5, 1, 4),        # padding beyond the picture on every side
    (16, 64, 46, 46, 128, 3, 3, 2, 1),     # 67 tiles of 128x128: 128x64 instead
    (127, 72, 16, 16, 136, 3, 3, 1, 1),    # 254 row tiles, two columns of 128: 508 tiles, the last of 8 channels
    (64, 100, 22, 22, 100, 3, 3, 1, 1),    # 242 tiles of 128: not enough
    (67, 100, 22, 22, 100, 3, 3, 1, 1),    # 254
    (68, 100, 22, 22, 100, 3, 3, 1, 1),    # 258
    (90, 128, 28, 28, 136, 3, 3, 2, 1),    # class pairs in 128x128 tiles
    (2, 20, 27, 30, 24, 4, 3, 2, 0),       # pairs of classes with unlike numbers of taps
    (3, 18, 12, 14, 40, 2, 1, 2, 0),       # ... none in some
    (2050, 24, 3, 3, 40, 3, 3, 1, 1),      # many small planes
]


@pytest.mark.parametrize("case", SHAPES)
def test_copied_tiles(case):
    q8t = require_gpu()
    od, (sx, px), (sw, pw), (sg, pg), _ = _conv_operands(synth.rng(sum(case)), case)
    d = q8t.conv_desc(*case)
    dpx, dpw, dpg = (qp_dev_from(p) for p in (px, pw, pg))
    oy, oacc = oracle.qconv_fwd(od, sx, px, sw, pw)
    y, acc = q8t.qconv_fwd(d, dev(sx), dpx, dev(sw), dpw, want_acc=True)
    same_ints(host(acc), oacc)
    same_ints(host(y), oy)
    odx, oacc = oracle.qconv_dgrad(od, sg, pg, sw, pw)
    dx, acc = q8t.qconv_dgrad(d, dev(sg), dpg, dev(sw), dpw, want_acc=True)
    same_ints(host(acc), oacc)
    same_ints(host(dx), odx)


FILTER_ROWS = [
    # N, C, H, W, K, R, S, stride, pad; the filter's rows (forward; layer gradient) and their mean bytes
    (2, 128, 5, 5, 40, 1, 1, 1, 0),        # 64 of 128: four a workgroup, just so
    (2, 129, 5, 5, 40, 1, 1, 1, 0),        # 64 of 144: one a workgroup
    (2, 128, 6, 6, 96, 3, 3, 4, 1),        # 2048 of 54, classes of 0 to 1 taps
    (3, 200, 9, 7, 72, 5, 5, 3, 2),        # 2304 of 222, channels of the last class beyond 200
    (1, 70, 13, 13, 512, 7, 7, 2, 3),      # 512 of 6272
    (2, 128, 9, 9, 128, 2, 2, 2, 0),       # 512 of 128, class pairs
    (2, 64, 9, 9, 128, 1, 1, 4, 0),        # 1024 of 8: a class with a tap, 15 without
]


@pytest.mark.parametrize("case", FILTER_ROWS)
def test_filter_rows_by_whole_workgroups_and_by_their_groups(case):
    test_copied_tiles(case)


def test_more_workgroups_than_one_dimension_of_a_launch_holds():
    # 16 stride classes of 2^26 planes of one position: 2^23 + 16 tiles of 512 threads, 2^32 threads and more
    import torch
    q8t = require_gpu()
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    N = (1 << 26) + 3
    d = q8t.conv_desc(N, 1, 1, 1, 1, 1, 1, 4, 0)
    assert q8t.qconv_workspace_size(d, 1) >= 16 * N      # the form with the channel-contiguous copy
    qg, pg = q8t.quantize(torch.randn((N, 1, 1, 1), device="cuda:0", generator=gen), 8)
    qw, pw = q8t.quantize(torch.full((1, 1, 1, 1), -0.7, device="cuda:0"), 8)
    dx, acc = q8t.qconv_dgrad(d, qg, pg, qw, pw, want_acc=True)
    zero = [int(p[4]) - 128 for p in (pg, pw)]
    want = (qg.int() - zero[0]) * (int(qw) - zero[1])
    assert torch.equal(acc, want)
    scale = torch.stack([p.view(torch.float32)[2] for p in (pg, pw)]).prod()
    assert torch.equal(dx, want.float() * scale)
