"""GPU parity of the wide-tile convolution kernel with few rows: tiles of 128, 64 and 32 rows, the last one short, filters packed
ahead for another batch size than the one that runs.  Bit-exact (integer accumulators, one rounding)."""
import pytest

import oracle
import synth
from gpu_util import close, dev, host, qp_dev_from, require_gpu, same_ints
from test_gpu_products import _conv_operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # N, C, H, W, K: 3x3, stride 1, pad 1
    (1, 64, 14, 14, 256),      # 32 rows, tiles of 4 columns in the last
    (1, 128, 7, 7, 128),       # ... no aligned groups of four, 128 columns in the filter's layout
    (3, 512, 7, 7, 256),       # ... 147 rows
    (5, 64, 9, 9, 384),
    (37, 64, 4, 4, 256),       # whole images inside a tile
    (24, 64, 14, 14, 256),     # 64 rows: 37 x 2 tiles of 128 x 128
    (47, 128, 7, 7, 512),      # ... 18.0 row tiles, the last one of 127 rows
    (50, 128, 9, 9, 384),      # ... 32 x 3
    (5, 64, 32, 32, 256),      # ... the widest plane
    (84, 64, 14, 14, 256),     # 128 rows: 129 x 2
])
def test_conv_few_rows(case):
    q8t = require_gpu()
    N, C, H, W, K = case
    case = (N, C, H, W, K, 3, 3, 1, 1)
    od, (sx, px), (sw, pw), (sg, pg), _ = _conv_operands(synth.rng(sum(case)), case)
    d = q8t.conv_desc(*case)
    dpx, dpw, dpg = (qp_dev_from(p) for p in (px, pw, pg))
    oy, oacc = oracle.qconv_fwd(od, sx, px, sw, pw)
    y, acc, stats = q8t.qconv_fwd_bn_stats(d, dev(sx), dpx, dev(sw), dpw, want_acc=True)
    same_ints(host(acc), oacc)
    same_ints(host(y), oy)
    yk = oy.astype("float64").transpose(1, 0, 2, 3).reshape(K, -1)
    close(host(stats)[0], yk.mean(axis=1))
    same_ints(host(stats)[1:], [yk.min(axis=1), yk.max(axis=1)])
    odx, oacc = oracle.qconv_dgrad(od, sg, pg, sw, pw)
    dx, acc = q8t.qconv_dgrad(d, dev(sg), dpg, dev(sw), dpw, want_acc=True)
    same_ints(host(acc), oacc)
    same_ints(host(dx), odx)


@pytest.mark.parametrize("channels", [256, 384])
def test_conv_filter_packed_for_another_batch(channels):
    q8t = require_gpu()
    small, large = (2, 128, 7, 7, channels, 3, 3, 1, 1), (600, 128, 7, 7, channels, 3, 3, 1, 1)
    od, (sx, px), (sw, pw), _, _ = _conv_operands(synth.rng(3), small)
    w = dev(sw)
    packed = q8t.qconv_pack_multi([(q8t.conv_desc(*large), 0, w)])[0]
    oy, _ = oracle.qconv_fwd(od, sx, px, sw, pw)
    y, _, _ = q8t.qconv_fwd_bn_stats(q8t.conv_desc(*small), dev(sx), qp_dev_from(px), w, qp_dev_from(pw), packed=packed)
    same_ints(host(y), oy)
