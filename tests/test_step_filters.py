"""The filters that a training step packs ahead are packed for the descriptors that its products use (CPU: the kernels are
replaced by functions that return tensors of the right shape and note what they were handed)."""
import pytest
import torch


@pytest.fixture
def step(monkeypatch):
    from test_abi import _lib_path
    _lib_path()
    from paper_1805_11046_amd import binding, train_step as ts
    made, products = {}, []

    def par():
        return torch.zeros(6, dtype=torch.int32)

    def codes(shape, dtype=torch.int8):
        return torch.zeros(shape, dtype=dtype), par()

    class Plan(binding.PackPlan):
        def run(self, qws, out=None):
            assert [tuple(q.shape) for q in qws] == self.shapes
            bufs = [torch.empty(s, dtype=torch.uint8) if s else None for s in self.sizes]
            for d, w, q, b in zip(self.descs, self.which, qws, bufs):
                if b is not None:
                    made[b.data_ptr()] = (bytes(d), w, q.data_ptr())
            return bufs

    def product(d, which, w, packed):
        size = binding.qconv_pack_size(d, which)
        products.append(size > 0)
        assert (packed is None) == (size == 0), (d.C, d.K, d.H, d.W, which)
        if size:
            assert made[packed.data_ptr()] == (bytes(d), which, w.data_ptr()), (d.C, d.K, d.H, d.W, which)

    def fwd(d, qx, px, qw, pw, packed=None):
        assert tuple(qx.shape) == (d.N, d.C, d.H, d.W) and tuple(qw.shape) == (d.K, d.C, d.R, d.S)
        if d.C != 3:
            product(d, 0, qw, packed)
        return torch.zeros((d.N, d.K, d.P, d.Q)), None, torch.zeros((3, d.K))

    def dgrad(d, g8, pg8, qw, pw, *more, packed=None):
        assert tuple(g8.shape) == (d.N, d.K, d.P, d.Q)
        product(d, 1, qw, packed)
        dx = torch.zeros((d.N, d.C, d.H, d.W))
        return dx if more else (dx, None)

    def bn_bwd(x, *a, want_dx=False, **k):
        return (torch.zeros_like(x), None, None) + codes(x.shape) + codes(x.shape, torch.int16)

    def pool(x, *a):
        shape = x.shape[:2] + tuple((v - 1) // 2 + 1 for v in x.shape[2:])
        return torch.zeros(shape), torch.zeros(shape, dtype=torch.uint8)

    for name, f in dict(
            PackPlan=Plan, quantize=lambda x, bits=8: codes(x.shape), quantize_multi=lambda t, bits: [codes(x.shape) for x in t],
            quantize_bifurcate=lambda g, *s: codes(g.shape) + codes(g.shape, torch.int16),
            qgemm_fwd=lambda x, px, w, pw: (torch.zeros(x.shape[0], w.shape[1]), None),
            qgemm_dgrad=lambda g, pg, w, pw: (torch.zeros(g.shape[0], w.shape[0]), None),
            qgemm_wgrad=lambda x, px, g, pg: (torch.zeros(x.shape[1], g.shape[1]), None),
            qconv_fwd_bn_stats=fwd, qconv_dgrad=dgrad, qconv_dgrad_relu_sum=dgrad, qconv_dgrad_sum=dgrad,
            qconv_wgrad=lambda d, *a, **k: (torch.zeros((d.K, d.C, d.R, d.S)), None),
            range_bn_bwd_bifurcate=bn_bwd, range_bn_relu_bwd_bifurcate=bn_bwd,
            maxpool_range_bn_bwd_bifurcate=lambda x, *a: bn_bwd(x)[1:],
            range_bn_bwd_bifurcate_masked=bn_bwd, range_bn_bwd_bifurcate_pass=bn_bwd,
            range_bn_relu_maxpool_fwd=pool, range_bn_relu_fwd_apply=lambda x, *a: (None,) + codes(x.shape),
            range_bn_add_relu_quantize=lambda x, *a, **k: (torch.zeros_like(x),) + codes(x.shape),
            range_bn_add_relu_pass=lambda x, *a, **k: (torch.zeros_like(x), None),
            relu_bwd_add=lambda g, *a: torch.zeros_like(g), relu_bwd_sum=lambda g, *a: torch.zeros_like(g),
            relu_bwd_sum_lattice=lambda g, *a: torch.zeros_like(g)).items():
        monkeypatch.setattr(binding, name, f)
    monkeypatch.setattr(ts, "_pack", True)
    ts._pack_plan.cache_clear()
    yield ts, products
    ts._pack_plan.cache_clear()


@pytest.mark.parametrize("batch,height,width", [(2, 64, 64), (2, 64, 160), (2, 160, 64), (2, 128, 96), (2, 96, 352),
                                                (2, 65, 131), (65, 32, 64), (300, 32, 32)])
def test_resnet18_products_take_filters_packed_for_their_own_descriptor(step, batch, height, width):
    ts, products = step
    ws = ts.make_weights(torch.device("cpu"), torch.Generator().manual_seed(0))
    ts.step(torch.zeros(batch, 3, height, width), torch.zeros(batch, dtype=torch.long), ws)
    assert len(products) == 2 * 19 and sum(products) >= 12


@pytest.mark.parametrize("height,width", [(14, 14), (5, 33), (56, 7)])
def test_bottleneck_products_take_filters_packed_for_their_own_descriptor(step, height, width):
    ts, products = step
    gen = torch.Generator().manual_seed(0)
    ws = [ts._he("cpu", gen, 64, 256, 1), ts._he("cpu", gen, 64, 64, 3), ts._he("cpu", gen, 256, 64, 1)]
    x = torch.zeros(2, 256, height, width, requires_grad=True)
    ts.bottleneck_step(x, torch.zeros(2, 256, height, width), ws)
    assert len(products) == 6


def test_weights_that_are_not_contiguous_are_refused_as_such(step, monkeypatch):
    from paper_1805_11046_amd import binding
    ts, _ = step

    def contiguous_only(t):
        if not t.is_contiguous():
            raise ValueError("q8t needs contiguous tensors")

    monkeypatch.undo()     # the calls check their own arguments, of CPU tensors too
    monkeypatch.setattr(binding, "_dev", contiguous_only)
    ws = [torch.zeros(c, k, r, r).transpose(0, 1) for k, c, r in ((64, 256, 1), (64, 64, 3), (256, 64, 1))]
    with pytest.raises(ValueError, match="contiguous"):
        ts.bottleneck_step(torch.zeros(2, 256, 14, 14, requires_grad=True), torch.zeros(2, 256, 14, 14), ws)


@pytest.mark.parametrize("bits", [False, True])
def test_bytes_booked_for_the_masked_backward_pass_are_those_it_moves(step, monkeypatch, bits):
    from paper_1805_11046_amd import binding
    ts, _ = step
    n, booked, call = 2 * 256 * 14 * 14, [], ts._call

    def note(name, ops, nbytes, fn, *a, **k):
        if name == "range_bn_bwd_bifurcate":     # the chain's last; those in front of it have the rectifier inside
            booked.append((nbytes, a[2].numel() * a[2].element_size()))
        return call(name, ops, nbytes, fn, *a, **k)

    monkeypatch.setattr(ts, "_call", note)
    if bits:
        monkeypatch.setattr(binding, "range_bn_bwd_bifurcate_masked", None)
        monkeypatch.setattr(binding, "range_bn_add_relu_pass",
                            lambda x, *a, **k: (torch.zeros_like(x), torch.zeros(x.numel() // 4, dtype=torch.uint8)))
    else:
        monkeypatch.setattr(binding, "range_bn_bwd_bifurcate_pass", None)
    gen = torch.Generator().manual_seed(0)
    ws = [ts._he("cpu", gen, 64, 256, 1), ts._he("cpu", gen, 64, 64, 3), ts._he("cpu", gen, 256, 64, 1)]
    ts.bottleneck_step(torch.zeros(2, 256, 14, 14, requires_grad=True), torch.zeros(2, 256, 14, 14), ws)
    # x and dy read, the masked gradient written and read, the two copies written; and what the mask comes from, once
    assert [nbytes for nbytes, _ in booked] == [(8 + 8 + 3) * n + by for _, by in booked] and len(booked) == 1
