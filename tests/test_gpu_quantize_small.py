"""GPU parity of the one-launch quantization of small tensors around its slices of 4096 elements and its limit: every
workgroup finds the range of the whole tensor, wherever its extremes lie."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host, require_gpu, same_ints, same_qparams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 1])      # 16-byte loads, single elements
@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 8188, 36864, 65533, 65536, 65537])
def test_small_tensors(n, off):
    q8t = require_gpu()
    x = synth.normal(synth.rng(n), (n,), std=1e-3)
    x[-1], x[n // 2] = 1.0, -2.0             # the range comes from other workgroups' slices
    buf = dev(np.concatenate([np.zeros(off, np.float32), x]))[off:]
    q, qp = q8t.quantize(buf, 8)
    s, _, oqp = oracle.quantize(x, 8)
    same_qparams(q8t, qp, oqp)
    same_ints(host(q), s)
    q8, p8, q16, p16 = q8t.quantize_bifurcate(buf, 7, 8)
    for bits, seed, got, gp in ((8, 7, q8, p8), (16, 8, q16, p16)):
        s, _, oqp = oracle.quantize(x, bits, stochastic=True, seed=seed)
        same_qparams(q8t, gp, oqp)
        same_ints(host(got), s)
        q, qp = q8t.quantize(buf, bits, stochastic=True, seed=seed)
        same_ints(host(q), s)
