"""The chained training step (paper_1805_11046_amd.train_step): the fused node structure (stem pooling inside the
Range BN pass, whole residual blocks as one node with the masked gradient sum, codes handed from layer to layer)
must give what the plain structure gives (every Range BN, ReLU, pooling, sum and quantization its own pass, torch's
autograd for the glue): same loss, same weight gradients.  Both run the same library products; a layer's stochastic
roundings are seeded by its position in the network, so the two structures draw the same random numbers."""
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def test_fused_and_plain_resnet18_steps_agree():
    require_gpu()
    import torch
    from paper_1805_11046_amd import train_step as ts
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    ws = ts.make_weights(dev, gen)
    x = torch.randn((4, 3, 224, 224), device=dev, generator=gen)
    labels = torch.randint(0, 1000, (4,), device=dev, generator=gen)
    params = [ws["conv1"], ws["fc"]] + [w for b in ws["blocks"] for w in b.values()]
    results = []
    for fuse in (True, False):
        ts._fuse = fuse
        for p in params:
            p.grad = None
        loss = ts.step(x, labels, ws)
        torch.cuda.synchronize()
        results.append((float(loss.detach()), [p.grad.clone() for p in params]))
    ts._fuse = True
    (lf, gf), (lp, gp) = results
    assert lf == lp
    for i, (a, b) in enumerate(zip(gf, gp)):
        assert torch.equal(a, b), "gradient of parameter %d differs: max |diff| %g" % (i, float((a - b).abs().max()))


def test_steps_leave_no_memory_behind():
    # the nodes of a step must not keep each other alive (a node that saves its own output would, until the cycle
    # collector happens to run): allocated device memory is the same after every step
    require_gpu()
    import gc
    import torch
    from paper_1805_11046_amd import train_step as ts
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(6)
    ws = ts.make_weights(dev, gen)
    x = torch.randn((2, 3, 224, 224), device=dev, generator=gen)
    labels = torch.randint(0, 1000, (2,), device=dev, generator=gen)
    params = [ws["conv1"], ws["fc"]] + [w for b in ws["blocks"] for w in b.values()]
    gc.collect()
    gc.disable()
    try:
        seen = []
        for _ in range(4):
            for p in params:
                p.grad = None
            ts.step(x, labels, ws)
            torch.cuda.synchronize()
            seen.append(torch.cuda.memory_allocated())
    finally:
        gc.enable()
    assert seen[1] == seen[2] == seen[3], seen


def test_weight_gradients_on_a_second_stream_change_nothing():
    require_gpu()
    import torch
    from paper_1805_11046_amd import train_step as ts
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(7)
    ws = ts.make_weights(dev, gen)
    x = torch.randn((4, 3, 224, 224), device=dev, generator=gen)
    labels = torch.randint(0, 1000, (4,), device=dev, generator=gen)
    params = [ws["conv1"], ws["fc"]] + [w for b in ws["blocks"] for w in b.values()]
    results = []
    try:
        for overlap in (False, True, True):
            ts._overlap = overlap
            for p in params:
                p.grad = None
            loss = ts.step(x, labels, ws)
            torch.cuda.synchronize()
            results.append((float(loss.detach()), [p.grad.clone() for p in params]))
    finally:
        ts._overlap = False
    for lo, go in results[1:]:
        assert lo == results[0][0]
        for i, (a, b) in enumerate(zip(results[0][1], go)):
            assert torch.equal(a, b), "gradient of parameter %d differs" % i


def test_filters_packed_in_one_launch_change_nothing():
    # the step with every filter packed ahead by one launch against the step whose products pack their own
    require_gpu()
    import torch
    from paper_1805_11046_amd import train_step as ts
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(11)
    ws = ts.make_weights(dev, gen)
    x = torch.randn((4, 3, 224, 224), device=dev, generator=gen)
    labels = torch.randint(0, 1000, (4,), device=dev, generator=gen)
    params = [ws["conv1"], ws["fc"]] + [w for b in ws["blocks"] for w in b.values()]
    results, before, lookup = [], ts._pack, ts._packed

    def counted(*a):
        b = lookup(*a)
        used.append(b is not None)
        return b

    ts._packed = counted
    try:
        for pack in (False, True, True):
            ts._pack, used = pack, []
            for p in params:
                p.grad = None
            loss = ts.step(x, labels, ws)
            torch.cuda.synchronize()
            results.append((float(loss.detach()), [p.grad.clone() for p in params]))
            assert len(used) == 38 and sum(used) == (30 if pack else 0)      # the products that have a packed form
            assert not ts._pcache
        with torch.no_grad():      # a weight that changes in place between two steps is packed anew
            ws["blocks"][4]["c2"].neg_()
        changed = []
        for pack in (False, True):
            ts._pack, used = pack, []
            for p in params:
                p.grad = None
            ts.step(x, labels, ws)
            torch.cuda.synchronize()
            changed.append([p.grad.clone() for p in params])
    finally:
        ts._pack, ts._packed = before, lookup
    assert not all(torch.equal(a, b) for a, b in zip(results[0][1], changed[0]))
    assert all(torch.equal(a, b) for a, b in zip(*changed))
    for lo, go in results[1:]:
        assert lo == results[0][0]
        for i, (a, b) in enumerate(zip(results[0][1], go)):
            assert torch.equal(a, b), "gradient of parameter %d differs" % i


def test_a_step_leaves_no_codes_behind():
    # a weight that changes in place after a step keeps its address: the next use has to quantize it again
    q8t = require_gpu()
    import torch
    from paper_1805_11046_amd import train_step as ts
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(7)
    ws = ts.make_weights(dev, gen)
    x = torch.randn((2, 3, 64, 64), device=dev, generator=gen)
    ts.step(x, torch.randint(0, 1000, (2,), device=dev, generator=gen), ws)
    a = torch.randn((8, 512), device=dev, generator=gen)
    with torch.no_grad():
        ws["fc"].mul_(-3.0)
        y = ts.Linear.apply(a, ws["fc"])
    (qa, pa), (qw, pw) = q8t.quantize(a, 8), q8t.quantize(ws["fc"].detach(), 8)
    assert torch.equal(y, q8t.qgemm_fwd(qa, pa, qw, pw)[0])


@pytest.mark.parametrize("height,width", [(64, 160), (256, 512), (128, 96)])
def test_filters_packed_ahead_change_nothing_on_oblong_images(height, width):
    # sizes at which the layout of a filter would be another one on a square image of either side
    require_gpu()
    import torch
    from paper_1805_11046_amd import train_step as ts
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(13)
    ws = ts.make_weights(dev, gen)
    x = torch.randn((2, 3, height, width), device=dev, generator=gen)
    labels = torch.randint(0, 1000, (2,), device=dev, generator=gen)
    params = [ws["conv1"], ws["fc"]] + [w for b in ws["blocks"] for w in b.values()]
    results, before = [], ts._pack
    try:
        for pack in (False, True):
            ts._pack = pack
            for p in params:
                p.grad = None
            loss = ts.step(x, labels, ws)
            torch.cuda.synchronize()
            results.append((float(loss.detach()), [p.grad.clone() for p in params]))
    finally:
        ts._pack = before
    assert results[0][0] == results[1][0]
    for i, (a, b) in enumerate(zip(results[0][1], results[1][1])):
        assert torch.equal(a, b), "gradient of parameter %d differs" % i
