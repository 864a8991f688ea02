"""A residual block as one node (train_step.Bottleneck): the pass that normalizes, adds the shortcut and rectifies, and the
layer gradient with the shortcut's gradient added in its epilogue, against the separate passes.  One rounding per fp32
operation on either side, so the results have to be the same bit for bit."""
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,mid,H", [
    (2, 256, 64, 56),    # register-tile kernel, 16-byte staging, fixed plane width
    (3, 128, 64, 20),    # ... any width
    (5, 256, 64, 14),    # ... 4-byte staging
    (2, 256, 64, 7),     # planes that are no multiple of 4: scalar pass, product and sum one after the other
    (2, 64, 16, 9),      # channel counts off 64: general kernels
])
def test_block_matches_separate_passes(N, C, mid, H):
    require_gpu()
    import torch
    from paper_1805_11046_amd import train_step as ts
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    ws = [ts._he(dev, gen, mid, C, 1), ts._he(dev, gen, mid, mid, 3), ts._he(dev, gen, C, mid, 1)]
    x = torch.randn((N, C, H, H), device=dev, generator=gen).abs_().requires_grad_(True)
    gy = torch.randn((N, C, H, H), device=dev, generator=gen) * 1e-3
    res = []
    try:
        for fuse in (True, False):
            ts._fuse = fuse
            for p in ws + [x]:
                p.grad = None
            out = ts.bottleneck_step(x, gy, ws)
            res.append([out.detach().clone()] + [p.grad.clone() for p in ws + [x]])
    finally:
        ts._fuse = True
    for i, (a, b) in enumerate(zip(*res)):
        assert torch.equal(a, b), "output %d differs: max |diff| %g" % (i, float((a - b).abs().max()))


@pytest.mark.parametrize("HW", [(8, 8), (5, 7)])
def test_block_tail_keeps_nan_and_inf(HW):
    q8t = require_gpu()
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(4)
    x = torch.randn((2, 6) + HW, device="cuda:0", generator=gen)
    o = torch.randn((2, 6) + HW, device="cuda:0", generator=gen)
    o[0, 1, 2, 3], o[1, 5, 4, 4], o[1, 0, 0, 0] = float("nan"), float("inf"), float("-inf")
    bn, stats, _, _ = q8t.range_bn_fwd(x, eps=1e-5)
    out = q8t.range_bn_add_relu(x, stats, o, eps=1e-5)
    assert torch.equal(torch.nan_to_num(out, nan=-1.0), torch.nan_to_num(torch.relu(bn + o), nan=-1.0))
