"""GPU parity of the FC products at the edges of their kernels' tiles: groups of four columns, pieces of 16 and steps of
64 of the reduction, splits of the reduction over wavefronts, the change to 128x128 tiles.  Accumulators bit-exact, float
results bit-exact as well (one or two roundings of an exact integer)."""
import pytest

import oracle
import synth
from gpu_util import dev, host, qp_dev_from, require_gpu, same_ints
from test_gpu_products import _rand_q

pytestmark = pytest.mark.gpu

SHAPES = [
    # M, N, K
    (16, 4, 16), (16, 16, 4), (17, 19, 18), (31, 66, 33), (33, 61, 64), (64, 64, 65),   # one tile, tails of all kinds
    (65, 130, 127), (96, 5, 300), (300, 7, 129), (257, 63, 513),                        # reductions split over 4 and 8 wavefronts
    (15, 40, 40), (40, 15, 15), (40, 3, 40), (40, 40, 3),                               # below the smallest piece: general kernel
    (600, 1800, 20), (1800, 20, 600), (20, 1800, 600), (523, 70, 66),                                  # more tiles than wavefronts to split
    (1500, 1410, 70), (1409, 66, 1502), (65, 1505, 1409), (1409, 1413, 64),             # 128x128 tiles, ragged in every direction
]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("off", [0, 1])
def test_fc_edges(M, N, K, off):
    q8t = require_gpu()
    if off and M * N * K > 20000000:
        pytest.skip("misaligned operands are covered at the small sizes")
    g = synth.rng(M * 7 + N * 3 + K)
    sx, px = _rand_q(g, (M, K))
    sw, pw = _rand_q(g, (K, N))
    sg, pg = _rand_q(g, (M, N))
    sg16, pg16 = _rand_q(g, (M, N), bits=16)
    dpx, dpw, dpg, dpg16 = (qp_dev_from(p) for p in (px, pw, pg, pg16))

    def put(a):   # off = 1: the operand starts one element behind an aligned address
        flat = dev(a.ravel())
        buf = flat.new_empty(flat.numel() + off)
        buf[off:] = flat
        return buf[off:].view(a.shape)

    y, acc = q8t.qgemm_fwd(put(sx), dpx, put(sw), dpw, want_acc=True)
    oy, oacc = oracle.qgemm_fwd(sx, px, sw, pw)
    same_ints(host(acc), oacc)
    same_ints(host(y), oy)
    dx, acc = q8t.qgemm_dgrad(put(sg), dpg, put(sw), dpw, want_acc=True)
    odx, oacc = oracle.qgemm_dgrad(sg, pg, sw, pw)
    same_ints(host(acc), oacc)
    same_ints(host(dx), odx)
    dw, acc = q8t.qgemm_wgrad(put(sx), dpx, put(sg16), dpg16, want_acc=True)
    odw, oacc = oracle.qgemm_wgrad(sx, px, sg16, pg16)
    same_ints(host(acc), oacc)
    same_ints(host(dw), odw)
