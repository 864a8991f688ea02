"""The C-ABI library loads without a GPU and exports every symbol the public header declares."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "q8t.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(q8t_[a-z0-9_]+)\s*\(", text)))


def _lib_path():
    path = os.path.join(ROOT, "paper_1805_11046_amd", "libq8t.so")
    if not os.path.exists(path):
        import __graft_entry__
        __graft_entry__.build()
    return path


def test_header_declares_the_expected_calls():
    names = _declared_functions()
    for must in ("q8t_quantize", "q8t_quantize_with_range", "q8t_quantize_bifurcate", "q8t_dequantize",
                 "q8t_qgemm_fwd", "q8t_qgemm_dgrad", "q8t_qgemm_wgrad", "q8t_qconv_fwd", "q8t_qconv_dgrad",
                 "q8t_qconv_wgrad", "q8t_range_bn_fwd", "q8t_range_bn_bwd", "q8t_range_bn_scale"):
        assert must in names


def test_library_exports_every_declared_symbol():
    lib = ctypes.CDLL(_lib_path())
    for name in _declared_functions():
        assert hasattr(lib, name), name


def test_binding_covers_every_declared_symbol():
    _lib_path()
    from paper_1805_11046_amd import binding
    assert sorted(binding.EXPORTED) == _declared_functions()


def test_host_only_calls():
    # these entry points do no GPU work: the closed form of Section 3 and size queries
    _lib_path()
    from paper_1805_11046_amd import binding
    import math
    assert binding.range_bn_scale(401408) == (2 * math.log(401408)) ** -0.5
    assert binding._lib.q8t_quantize_workspace_size(1 << 20) >= 8
    d = binding.conv_desc(128, 64, 56, 56, 64, 3, 3, 1, 1)
    assert (d.P, d.Q) == (56, 56)
    for which in (0, 1, 2):
        assert binding._lib.q8t_qconv_workspace_size(ctypes.byref(d), which) >= 0
    # the first layer of a ResNet at batch 256 runs on the kernel that builds its operand in LDS: its workspace is
    # the packed filter, not 630 MB of explicit im2col rows
    d1 = binding.conv_desc(256, 3, 224, 224, 64, 7, 7, 2, 3)
    assert 0 < binding._lib.q8t_qconv_workspace_size(ctypes.byref(d1), 0) < (1 << 20)
    assert "gfx950" in binding.version()


def test_argument_errors_are_reported_before_any_launch():
    _lib_path()
    from paper_1805_11046_amd import binding
    L = binding._lib
    assert L.q8t_quantize(None, 16, 8, 0, 0, None, None, None, None) == -1      # NULL
    assert L.q8t_quantize(None, -1, 8, 0, 0, None, None, None, None) == -2      # shape
    assert L.q8t_quantize(None, 16, 17, 0, 0, None, None, None, None) == -3     # bits
    assert L.q8t_quantize_noalloc(None, (1 << 34) + 1, 8, 0, 0, None, None, None) == -2   # beyond the maximum
    assert L.q8t_quantize_noalloc(None, 16, 8, 0, 0, None, None, None) == -1
    assert L.q8t_qgemm_fwd(None, None, None, None, 0, 1, 1, None, None, None, None) == -2
    assert L.q8t_range_bn_fwd(None, 1, 1, 1, 1, None, None, 0.0, None, None, None, None, None, None) == -2


def test_packed_filter_sizes_follow_the_kernel_that_serves_the_shape():
    # host logic of the packed filters: codes rounded up to 256 bytes + one column sum per output channel of the product,
    # for the shapes the register-tile and wide-tile kernels take; nothing for the others
    _lib_path()
    from paper_1805_11046_amd import binding

    def size(case, which):
        return binding.qconv_pack_size(binding.conv_desc(*case), which)

    def expect(case, which):
        n, c, h, w, k, r, s, st, pad = case
        up = lambda v: (v + 255) // 256 * 256
        return up(k * c * r * s) + up(4 * (k if which == 0 else c))

    for case in ((256, 256, 14, 14, 256, 3, 3, 1, 1), (256, 512, 7, 7, 512, 3, 3, 1, 1), (256, 64, 56, 56, 64, 3, 3, 1, 1),
                 (8, 64, 28, 28, 128, 1, 1, 1, 0)):
        for which in (0, 1):
            assert size(case, which) == expect(case, which)
    lattice = (256, 64, 56, 56, 128, 1, 1, 2, 0)       # forward on the gathered positions; its layer gradient packs nothing
    assert size(lattice, 0) == expect(lattice, 0) and size(lattice, 1) == 0
    for case in ((256, 64, 56, 56, 128, 3, 3, 2, 1), (256, 3, 224, 224, 64, 7, 7, 2, 3), (2, 3, 7, 6, 4, 3, 3, 1, 1)):
        assert size(case, 0) == 0 and size(case, 1) == 0
    assert size(lattice, 2) == 0                       # the weight gradient reads no filter
    L = binding._lib
    assert L.q8t_qconv_pack_multi(1, None, None, None, None, None) == -1
    assert L.q8t_qconv_pack_multi(0, None, None, None, None, None) == 0


def test_long_reductions_under_few_results_are_split():
    # slices of the reduction in workgroups of their own leave their partial results in the workspace
    _lib_path()
    from paper_1805_11046_amd import binding
    size = binding._lib.q8t_qgemm_workspace_size
    for M, N, K, which in ((65536, 64, 64, 2), (64, 64, 16384, 0), (61, 29390, 29, 1)):
        assert size(M, N, K, which) >= 2 * 8 * {0: M * N, 1: M * K, 2: K * N}[which]
    assert size(256, 1000, 512, 0) == 0


def test_form_of_a_product_follows_its_size():
    # the workspace shows which form serves a shape that no specialised kernel takes
    _lib_path()
    from paper_1805_11046_amd import binding

    def size(*case):
        return binding.qconv_workspace_size(binding.conv_desc(*case), 0)

    assert size(56, 3, 7, 7, 64, 1, 1, 1, 0) == 0                             # general kernel: one launch, no workspace
    rows = 5 * 7 * 4
    assert size(5, 472, 7, 4, 1, 7, 7, 1, 3) % (8 * rows) == 0                # general kernel, slices of int64 results
    assert 0 < size(40, 16, 32, 32, 16, 3, 3, 1, 1) - 40 * 32 * 32 * 16 < 1 << 17   # copy of the operand, packed filter, tables
    assert 0 < size(64, 32, 27, 27, 512, 1, 1, 1, 0) - 64 * 27 * 27 * 32 < 1 << 17
    assert 0 < size(64, 3, 27, 27, 64, 7, 7, 2, 3) - 64 * 27 * 27 * 16 < 1 << 17   # 13.0 us; first-layer kernel 14.7
    assert 64 * 64 <= size(128, 1, 56, 56, 64, 5, 5, 1, 2) < 1 << 16          # first-layer kernel (28 us; copy 56): the packed filter
    assert 0 < size(256, 3, 28, 28, 512, 7, 7, 2, 3) - 256 * 14 * 14 * 192 < 1 << 18   # im2col rows: 147 columns filled up to 192


@pytest.mark.parametrize("case", [(6, 496, 27, 4, 4, 1, 1, 4, 0), (111, 42, 17, 17, 3, 1, 1, 2, 0),    # 8.6 us, copied 14.1; 9.9, 15.8
                                  (367, 56, 9, 9, 4, 2, 2, 2, 1), (3510, 256, 5, 5, 7, 1, 1, 2, 0)])   # 13.3, 21.4; 64, 157
def test_layer_gradients_of_few_channels_to_scattered_results_need_no_copy(case):
    _lib_path()
    from paper_1805_11046_amd import binding
    assert binding.qconv_workspace_size(binding.conv_desc(*case), 1) == 0     # general kernel


def test_weight_gradient_of_a_filter_as_large_as_the_plane_lays_out_no_padding():
    # one result a plane: 1024 positions of the gradient's byte planes and the codes once, beside the partial tiles
    _lib_path()
    from paper_1805_11046_amd import binding
    K, crs, positions = 512, 512 * 49, 1024
    size = binding.qconv_workspace_size(binding.conv_desc(positions, 512, 7, 7, K, 7, 7, 1, 0), 2)
    tiles = 2 * K * crs * 4
    assert tiles < size < tiles + (2 * K + crs) * positions + (4 << 20)
