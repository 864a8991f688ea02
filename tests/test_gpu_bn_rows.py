"""GPU parity of Range BN over FC activations ([N][C], planes of one position): column blocks of 8, 16 and 32 with and
without a remainder, fewer rows than a workgroup takes at a time and more, ties of the extrema, the codes' route, and the
plane kernels behind the limit of rows."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import close, dev, host, require_gpu, same_ints, same_qparams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("affine", [False, True])
@pytest.mark.parametrize("N,C", [(2, 1), (2, 8), (64, 128), (127, 9), (129, 511), (63, 512), (65, 527), (70, 2047), (31, 2048),
                                 (33, 2049), (2048, 17), (2049, 17),
                                 (4096, 1030), (4097, 1024)])
def test_range_bn_over_rows(N, C, affine):
    q8t = require_gpu()
    g = synth.rng(N + C)
    x = np.round(synth.normal(g, (N, C, 1, 1), std=20.0)) / 8      # a coarse grid: extrema attained more than once
    dy = synth.normal(g, (N, C, 1, 1), std=1e-2)
    ga = be = None
    if affine:
        ga, be = 1 + synth.normal(g, (C,), std=0.1), synth.normal(g, (C,), std=0.1)
    x, dy = x.astype(np.float32), dy.astype(np.float32)
    ga, be = (None if v is None else v.astype(np.float32) for v in (ga, be))
    dga, dbe = (None if v is None else dev(v) for v in (ga, be))
    y, stats, _, _ = q8t.range_bn_fwd(dev(x), dga, dbe, 1e-5)
    oy, ost, _, _ = oracle.range_bn_fwd(x, ga, be, 1e-5)
    st = host(stats)
    close(st[0], ost[0])
    same_ints(st[1:], ost[1:])
    close(host(y), oy)
    yq, sq, q, qp = q8t.range_bn_fwd(dev(x), dga, dbe, 1e-5, quantized=True)
    same_ints(host(sq), st)
    same_ints(host(yq), host(y))
    codes, cp = q8t.quantize(y, 8)
    same_ints(host(q), host(codes))
    assert q8t.qparams_to_host(qp) == q8t.qparams_to_host(cp)
    dx, dg, db = q8t.range_bn_bwd(dev(x), dev(dy), stats, dga, 1e-5)
    odx, odg, odb = oracle.range_bn_bwd(x, dy, st, ga, 1e-5)
    close(host(dx), odx)
    close(host(dg), odg)
    close(host(db), odb)
