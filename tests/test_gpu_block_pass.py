"""The bits that the tail of a residual block leaves for its backward pass: the same results as with the block's result itself,
with float4 and with single accesses, planes smaller and larger than a workgroup's sweep, NaN and infinities in the sum."""
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2, 6, 8, 8), (3, 5, 2, 2), (5, 7, 36, 36), (2, 3, 64, 66), (70, 9, 10, 14)])
@pytest.mark.parametrize("aligned", [True, False])
def test_bits_for_the_backward_pass(shape, aligned):
    q8t = require_gpu()
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(sum(shape))
    x = torch.randn(shape, device="cuda:0", generator=gen)
    o = torch.randn(shape, device="cuda:0", generator=gen)
    o.view(-1)[:3] = torch.tensor([float("nan"), float("inf"), float("-inf")])
    stats = q8t.range_bn_fwd(x, eps=1e-5)[1]
    out, bits = q8t.range_bn_add_relu_pass(x, stats, o, eps=1e-5)
    expected = q8t.range_bn_add_relu(x, stats, o, eps=1e-5)
    assert torch.equal(out.view(torch.int32), expected.view(torch.int32))
    assert bits.dtype == torch.uint8 and bits.numel() * 4 == x.numel()
    passes = ~(out <= 0).view(-1, 4)
    assert torch.equal(bits, (passes * torch.tensor([1, 2, 4, 8], device="cuda:0")).sum(1).to(torch.uint8))
    flat = torch.randn(x.numel() + 1, device="cuda:0", generator=gen)
    dy = (flat[:-1] if aligned else flat[1:]).view(shape)
    a = q8t.range_bn_bwd_bifurcate_masked(x, dy, out, stats, None, 1e-5, 3, 4)
    b = q8t.range_bn_bwd_bifurcate_pass(x, dy, bits, stats, None, 1e-5, 3, 4)
    for s, t in zip(a, b):
        assert torch.equal(s, t)


def test_no_bits_where_four_elements_are_no_unit():
    q8t = require_gpu()
    import torch
    x = torch.randn((2, 6, 5, 7), device="cuda:0")
    stats = q8t.range_bn_fwd(x, eps=1e-5)[1]
    out, bits = q8t.range_bn_add_relu_pass(x, stats, x, eps=1e-5)
    assert bits is None and torch.equal(out, q8t.range_bn_add_relu(x, stats, x, eps=1e-5))
    flat = torch.randn(2 * 6 * 8 * 8 + 1, device="cuda:0")
    y = torch.randn((2, 6, 8, 8), device="cuda:0")
    assert q8t.range_bn_add_relu_pass(y, q8t.range_bn_fwd(y, eps=1e-5)[1], flat[1:].view(y.shape), eps=1e-5)[1] is None
