"""GPU parity of the general weight gradient on padded planes: pads shared between rows and images or not, one input plane
per stride class, groups of four positions across rows, images and the end of a tensor, tiles of rows and columns with a
remainder, several groups of wavefronts on a tile.  Bit-exact (integer sums)."""
import pytest

import oracle
import synth
from gpu_util import dev, host, qp_dev_from, require_gpu, same_ints
from test_gpu_products import _conv_operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # N, C, H, W, K, R, S, stride, pad
    (5, 96, 27, 27, 200, 3, 3, 1, 1),     # pads shared by rows and images; 400 rows, 864 columns
    (40, 16, 32, 32, 16, 3, 3, 1, 1),     # fewer rows than a tile
    (9, 17, 33, 31, 47, 3, 3, 1, 1),
    (60, 65, 15, 14, 129, 3, 3, 1, 1),    # one row and 71 columns behind a tile
    (3, 24, 36, 36, 40, 7, 7, 1, 3),
    (3, 24, 36, 37, 40, 7, 5, 1, 1),      # less padding than the filter's reach
    (3, 24, 36, 37, 40, 5, 5, 1, 0),      # none
    (4, 40, 35, 33, 72, 3, 3, 2, 1),      # four input planes a channel
    (6, 80, 30, 28, 48, 1, 1, 2, 0),      # one of them read
    (7, 80, 29, 27, 48, 1, 1, 1, 0),      # no pads at all, 783 positions
    (3, 36, 40, 40, 50, 5, 4, 3, 2),
    (5, 20, 41, 43, 24, 3, 3, 5, 1),      # stride beyond the filter
    (5, 20, 41, 43, 24, 7, 6, 4, 5),      # more padding than a stride
    (300, 48, 5, 5, 63, 3, 3, 1, 1),      # 36 positions for 25
    (700, 33, 2, 3, 40, 2, 1, 1, 0),      # groups of four over three images
    (900, 70, 1, 1, 65, 1, 1, 1, 0),      # ... over four
    (400, 48, 3, 3, 63, 3, 3, 1, 1),      # 16 positions for 9
    (400, 48, 2, 2, 63, 3, 3, 1, 1),      # 9 for 4
    (100, 16, 4, 4, 40, 7, 7, 1, 3),      # 49 for 16
    (100, 128, 14, 14, 128, 5, 5, 1, 2),  # 256x256 tiles of byte planes; columns 3200
    (260, 130, 20, 20, 4, 3, 3, 1, 1),    # several slices, one row tile
    (1, 3, 300, 280, 5, 5, 5, 1, 2),
])
def test_weight_gradient_padded(case):
    q8t = require_gpu()
    od, (sx, px), _, _, (s16, p16) = _conv_operands(synth.rng(sum(case)), case)
    odw, oacc = oracle.qconv_wgrad(od, sx, px, s16, p16)
    d = q8t.conv_desc(*case)
    dw, acc = q8t.qconv_wgrad(d, dev(sx), qp_dev_from(px), dev(s16), qp_dev_from(p16), want_acc=True)
    same_ints(host(acc), oacc)
    same_ints(host(dw), odw)


def test_weight_gradient_padded_at_odd_addresses():
    import torch
    q8t = require_gpu()
    case = (6, 33, 15, 16, 50, 3, 3, 1, 1)
    od, (sx, px), _, _, (s16, p16) = _conv_operands(synth.rng(5), case)
    _, oacc = oracle.qconv_wgrad(od, sx, px, s16, p16)
    x, g = dev(sx), dev(s16)
    for off in (1, 2, 3):
        bx = torch.empty(x.numel() + off, dtype=torch.int8, device=x.device)
        bg = torch.empty(g.numel() + off, dtype=torch.int16, device=x.device)
        x2, g2 = bx[off:].view(x.shape), bg[off:].view(g.shape)
        x2.copy_(x)
        g2.copy_(g)
        _, acc = q8t.qconv_wgrad(q8t.conv_desc(*case), x2, qp_dev_from(px), g2, qp_dev_from(p16), want_acc=True)
        same_ints(host(acc), oacc)
