"""The native call module: what it refuses before any device work (CPU)."""
import pytest
import torch


@pytest.fixture(scope="module")
def q8t():
    from test_abi import _lib_path
    _lib_path()
    import paper_1805_11046_amd as m
    return m


def test_cpu_tensors_are_refused(q8t):
    x = torch.zeros(8, 8)
    i8, p = torch.zeros(8, 8, dtype=torch.int8), torch.zeros(6, dtype=torch.int32)
    d = q8t.conv_desc(1, 1, 8, 8, 1, 3, 3, 1, 1)
    for call in (lambda: q8t.quantize(x), lambda: q8t.quantize_bifurcate(x), lambda: q8t.quantize_with_range(x, x),
                 lambda: q8t.qgemm_fwd(i8, p, i8, p), lambda: q8t.qgemm_dgrad(i8, p, i8, p), lambda: q8t.qgemm_wgrad(i8, p, i8, p),
                 lambda: q8t.qconv_fwd_bn_stats(d, i8, p, i8, p), lambda: q8t.qconv_dgrad(d, i8, p, i8, p),
                 lambda: q8t.qconv_wgrad(d, i8, p, i8, p), lambda: q8t.range_bn_fwd(x), lambda: q8t.range_bn_bwd(x, x, x),
                 lambda: q8t.range_bn_relu_fwd_apply(x, x), lambda: q8t.range_bn_relu_bwd_bifurcate(x, x, x),
                 lambda: q8t.range_bn_bwd_bifurcate(x, x, x), lambda: q8t.range_bn_add_relu_quantize(x, x, x),
                 lambda: q8t.chunk_range(x, 4), lambda: q8t.qconv_dgrad_relu_sum(d, i8, p, i8, p, x, x),
                 lambda: q8t.qconv_dgrad_sum(d, i8, p, i8, p, x), lambda: q8t.range_bn_bwd_bifurcate_masked(x, x, x, x)):
        with pytest.raises(ValueError, match="device tensors only"):
            call()


def test_other_arguments_than_tensors_are_refused(q8t):
    for call in (lambda: q8t.quantize([1.0]), lambda: q8t.qgemm_fwd(None, None, None, None),
                 lambda: q8t.qconv_wgrad(3, None, None, None, None)):
        with pytest.raises((TypeError, AttributeError)):
            call()
