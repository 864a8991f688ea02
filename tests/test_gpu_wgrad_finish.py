"""GPU parity of the weight gradient on padded planes where its last step (partial sums of the image ranges -> dW) changes
its split: one, two, four or eight groups of lanes, filters of one and of nine taps, one range up to many.  Bit-exact."""
import pytest

import oracle
import synth
from gpu_util import dev, host, qp_dev_from, require_gpu, same_ints
from test_gpu_products import _conv_operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (3, 64, 14, 14, 64, 1, 1, 2, 0),      # one tap, one range: one group
    (7, 64, 14, 14, 64, 1, 1, 2, 0),      # ... two ranges: two groups
    (50, 64, 14, 14, 64, 1, 1, 2, 0),     # ... thirteen ranges: more than wavefronts
    (9, 256, 14, 14, 256, 1, 1, 2, 0),    # ... 16 tiles, three ranges
    (9, 512, 14, 14, 256, 1, 1, 2, 0),    # ... 32 tiles: one group, three ranges
    (4, 64, 7, 7, 64, 3, 3, 1, 1),        # nine taps, one range
    (5, 64, 7, 7, 64, 3, 3, 1, 1),        # ... two
    (2, 64, 56, 56, 128, 3, 3, 2, 1),     # ... planes in bands
    (16, 64, 14, 14, 64, 3, 3, 1, 1),     # ... one tile, sixteen ranges: eight groups
    (83, 64, 14, 14, 64, 3, 3, 2, 1),     # ... 21 ranges, no multiple of the groups
    (70, 64, 28, 28, 64, 3, 3, 2, 1),     # ... 70 ranges
    (1, 512, 14, 14, 512, 1, 1, 2, 0),    # one tap, one range, 64 tiles
    (9, 256, 14, 14, 512, 3, 3, 2, 1),    # nine taps, 32 tiles, three ranges, the last chunk incomplete
])
def test_weight_gradient_finish(case):
    q8t = require_gpu()
    od, (sx, px), _, _, (s16, p16) = _conv_operands(synth.rng(sum(case)), case)
    odw, oacc = oracle.qconv_wgrad(od, sx, px, s16, p16)
    dw, acc = q8t.qconv_wgrad(q8t.conv_desc(*case), dev(sx), qp_dev_from(px), dev(s16), qp_dev_from(p16), want_acc=True)
    same_ints(host(acc), oacc)
    same_ints(host(dw), odw)
