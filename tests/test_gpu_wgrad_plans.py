"""GPU parity of the general weight gradient in each of its plans: padded planes or a plane of the input per tap (through LDS where a
plane has one to three results), with and without groups of wavefronts that share a tile.  Bit-exact."""
import pytest

import oracle
import synth
from gpu_util import dev, host, qp_dev_from, require_gpu, same_ints
from test_gpu_products import _conv_operands

pytestmark = pytest.mark.gpu

SHAPES = [
    # N, C, H, W, K, R, S, stride, pad
    (300, 40, 1, 1, 50, 1, 1, 1, 0),       # one result a plane: 64 images a group and a remainder
    (1001, 33, 5, 5, 12, 5, 5, 1, 0),      # ... under a filter as large as the plane
    (70, 70, 7, 7, 72, 7, 7, 1, 0),
    (301, 33, 1, 2, 50, 1, 1, 1, 0),       # two results
    (259, 40, 3, 1, 20, 3, 3, 1, 1),       # three, padded
    (123, 40, 2, 2, 33, 3, 3, 2, 1),       # a stride
    (2, 300, 4, 4, 200, 4, 4, 1, 0),       # fewer images than a dword has positions
    (77, 40, 6, 5, 24, 4, 4, 1, 0),        # a plane per tap with six results: rows of positions shorter than rows of codes
    (64, 48, 8, 8, 96, 6, 6, 1, 0),
    (90, 24, 9, 10, 30, 8, 7, 2, 0),
    (18, 150, 12, 12, 300, 3, 3, 1, 1),    # tiles just above the number of compute units: no groups
    (16, 64, 30, 30, 40, 5, 5, 1, 2),      # few tiles: groups
]


@pytest.mark.parametrize("case", SHAPES)
def test_weight_gradient_plans(case):
    q8t = require_gpu()
    od, (sx, px), _, _, (sg, pg) = _conv_operands(synth.rng(sum(case)), case)
    d = q8t.conv_desc(*case)
    dw, acc = q8t.qconv_wgrad(d, dev(sx), qp_dev_from(px), dev(sg), qp_dev_from(pg), want_acc=True)
    odw, oacc = oracle.qconv_wgrad(od, sx, px, sg, pg)
    same_ints(host(acc), oacc)
    same_ints(host(dw), odw)
