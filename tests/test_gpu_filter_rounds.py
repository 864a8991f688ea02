"""GPU parity of products whose filter is packed in several rounds of 256 reduction channels, the last one short: every layout,
both directions, packed by the product itself and ahead.  Bit-exact (integer accumulators, one rounding)."""
import pytest

import oracle
import synth
from gpu_util import dev, host, qp_dev_from, require_gpu, same_ints
from test_gpu_products import _conv_operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (1, 320, 8, 8, 576, 3, 3, 1, 1),     # 64-column layout: rounds of 256 + 64 forward, 256 + 256 + 64 backward
    (2, 832, 4, 4, 384, 3, 3, 1, 1),     # 128 columns forward, 64 backward
    (1, 640, 7, 7, 768, 3, 3, 1, 1),     # 256 columns forward, 128 backward
    (3, 576, 4, 4, 320, 1, 1, 1, 0),     # 1x1
    (1, 64, 6, 6, 1088, 1, 1, 1, 0),
])
def test_conv_filter_of_several_rounds(case):
    q8t = require_gpu()
    od, (sx, px), (sw, pw), (sg, pg), _ = _conv_operands(synth.rng(sum(case)), case)
    d, w = q8t.conv_desc(*case), dev(sw)
    dpx, dpw, dpg = (qp_dev_from(p) for p in (px, pw, pg))
    oy, oacc = oracle.qconv_fwd(od, sx, px, sw, pw)
    odx, odacc = oracle.qconv_dgrad(od, sg, pg, sw, pw)
    ahead = q8t.qconv_pack_multi([(d, 0, w), (d, 1, w)])
    assert all(b is not None for b in ahead)
    for packed in ((None, None), ahead):
        y, acc, _ = q8t.qconv_fwd_bn_stats(d, dev(sx), dpx, w, dpw, want_acc=True, packed=packed[0])
        same_ints(host(acc), oacc)
        same_ints(host(y), oy)
        dx, acc = q8t.qconv_dgrad(d, dev(sg), dpg, w, dpw, want_acc=True, packed=packed[1])
        same_ints(host(acc), odacc)
        same_ints(host(dx), odx)
