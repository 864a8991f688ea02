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


# 128x128 tiles whose reduction is longer than the two steps of prefetch: odd and even numbers of steps, with a last piece
# that reaches back and without, operands at odd addresses and of odd pitch
@pytest.mark.parametrize("which", ["fwd", "dgrad", "wgrad"])
@pytest.mark.parametrize("red,off", [(129, 0), (192, 0), (300, 0), (320, 1), (333, 0), (333, 1), (384, 0), (1025, 0)])
def test_fc_tile_pipeline(which, red, off):
    q8t = require_gpu()
    R, Cc = 1409, 1411
    g = synth.rng(red)

    def put(a):
        flat = dev(a.ravel())
        buf = flat.new_empty(flat.numel() + off)
        buf[off:] = flat
        return buf[off:].view(a.shape)

    shapes = {"fwd": ((R, red), (red, Cc)), "dgrad": ((R, red), (Cc, red)), "wgrad": ((red, R), (red, Cc))}[which]
    a, pa = _rand_q(g, shapes[0])
    b, pb = _rand_q(g, shapes[1], **({"bits": 16} if which == "wgrad" else {}))
    out, acc = getattr(q8t, "qgemm_" + which)(put(a), qp_dev_from(pa), put(b), qp_dev_from(pb), want_acc=True)
    oout, oacc = getattr(oracle, "qgemm_" + which)(a, pa, b, pb)
    same_ints(host(acc), oacc)
    same_ints(host(out), oout)


# few results under a long reduction: slices of it in workgroups of their own, the last one shorter, pieces that reach back
# into the slice before, results that hang over the edge of a tile
@pytest.mark.parametrize("M,N,K", [
    (7, 5, 2047), (7, 5, 2048), (6, 5, 27421), (33, 70, 4097), (16, 4096, 4100), (65, 66, 16400), (480, 260, 9000),   # forward
    (5, 2049, 6), (61, 29390, 29), (96, 5000, 130), (1607, 8229, 14),                                                 # layer gradient
    (2047, 9, 34), (2065, 12, 237), (65535, 4, 5), (65536, 70, 19), (4101, 600, 195), (8300, 70, 515),                # weight gradient
])
def test_fc_split_reduction(M, N, K):
    test_fc_edges(M, N, K, 0)


# one K-step: tiles shared by more wavefronts than it has steps, narrow results, and the general kernel's range
@pytest.mark.parametrize("M,N,K", [(16, 16, 16), (64, 1000, 1000), (64, 1025, 1030), (64, 9000, 70), (4001, 1000, 40), (1000, 40, 4000), (64, 16, 17000)])
def test_fc_single_step(M, N, K):
    test_fc_edges(M, N, K, 0)


def test_fc_split_needs_its_workspace():
    q8t = require_gpu()
    import torch
    x, w = torch.zeros((8, 8192), dtype=torch.int8, device="cuda:0"), torch.zeros((8192, 8), dtype=torch.int8, device="cuda:0")
    _, px = q8t.quantize(torch.zeros(4, device="cuda:0"), 8)
    with pytest.raises(q8t.Q8TError) as e:
        q8t.binding._check(q8t.binding._lib.q8t_qgemm_fwd(x.data_ptr(), px.data_ptr(), w.data_ptr(), px.data_ptr(), 8, 8, 8192,
                                                          x.data_ptr(), None, None, 0), "q8t_qgemm_fwd")
    assert e.value.code == -5


# tiles that go to LDS without registers: rows of whole 16-byte pieces, many tiles; the reduction in one step, in whole steps,
# with a tail of one or several pieces (forward: of both operands; otherwise any length along slow indices), rows and columns
# that end inside a tile, the first sizes that go this way, and neighbours that do not
@pytest.mark.parametrize("which,R,Cc,red", [
    ("fwd", 1409, 1424, 80), ("fwd", 1409, 1424, 128), ("fwd", 1537, 1296, 144), ("fwd", 1409, 1424, 1040), ("fwd", 4000, 400, 272),
    ("fwd", 1025, 1152, 1024), ("fwd", 1025, 1152, 1008), ("fwd", 16384, 96, 64), ("fwd", 16384, 80, 64),
    ("dgrad", 1409, 1413, 80), ("dgrad", 1537, 1283, 256), ("dgrad", 1409, 1411, 400), ("dgrad", 100, 16390, 64), ("dgrad", 129, 8193, 1040),
    ("wgrad", 1424, 1000, 64), ("wgrad", 1040, 808, 127), ("wgrad", 1040, 808, 128), ("wgrad", 1536, 776, 129), ("wgrad", 1424, 584, 300),
    ("wgrad", 112, 7168, 1027), ("wgrad", 16400, 48, 65),
    ("wgrad", 1296, 808, 127), ("wgrad", 1296, 808, 128), ("wgrad", 1424, 776, 300), ("wgrad", 112, 8448, 1027),
    ("wgrad", 1024, 1024, 1030), ("wgrad", 1040, 1024, 1030),      # 256 tiles of 64x64: not copied; 272
])
def test_fc_copied_tiles(which, R, Cc, red):
    q8t = require_gpu()
    g = synth.rng(R + 3 * Cc + red)
    M, N, K = {"fwd": (R, Cc, red), "dgrad": (R, red, Cc), "wgrad": (red, Cc, R)}[which]
    if which == "fwd":
        (sa, pa), (sb, pb) = _rand_q(g, (M, K)), _rand_q(g, (K, N))
        out, want = q8t.qgemm_fwd, oracle.qgemm_fwd
    elif which == "dgrad":
        (sa, pa), (sb, pb) = _rand_q(g, (M, N)), _rand_q(g, (K, N))
        out, want = q8t.qgemm_dgrad, oracle.qgemm_dgrad
    else:
        (sa, pa), (sb, pb) = _rand_q(g, (M, K)), _rand_q(g, (M, N), bits=16)
        out, want = q8t.qgemm_wgrad, oracle.qgemm_wgrad
    y, acc = out(dev(sa), qp_dev_from(pa), dev(sb), qp_dev_from(pb), want_acc=True)
    oy, oacc = want(sa, pa, sb, pb)
    same_ints(host(acc), oacc)
    same_ints(host(y), oy)
