"""Calls on several streams and in graphs, with the workspaces that the Python calls take by themselves."""
import pytest

import synth
from gpu_util import dev, qp_dev_from, require_gpu
from test_gpu_products import _conv_operands

pytestmark = pytest.mark.gpu

# both keep a copy of their operand, the reordered filter and tables in the workspace, at different places
CASES = [(24, 40, 30, 30, 72, 3, 3, 1, 1), (30, 72, 24, 26, 200, 3, 3, 2, 1)]


def _calls(q8t):
    calls = []
    for case in CASES:
        _, (sx, px), (sw, pw), (sg, pg), _ = _conv_operands(synth.rng(sum(case)), case)
        d, args = q8t.conv_desc(*case), [dev(sx), qp_dev_from(px), dev(sw), qp_dev_from(pw), dev(sg), qp_dev_from(pg)]
        calls.append(lambda d=d, a=args: (q8t.qconv_fwd(d, *a[:4])[0], q8t.qconv_dgrad(d, a[4], a[5], a[2], a[3])[0]))
    return calls


def test_two_streams():
    q8t = require_gpu()
    import torch
    calls = _calls(q8t)
    expected = [c() for c in calls]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in calls]
    for _ in range(8):
        got = []
        for s, c in zip(streams, calls):
            s.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(s):
                got.append([c() for _ in range(3)])
        torch.cuda.synchronize()
        for e, rounds in zip(expected, got):
            for r in rounds:
                assert all(torch.equal(x, y) for x, y in zip(r, e))


def test_graph_keeps_its_workspace():
    # a larger call between the replays makes the kept buffer grow and the old one go back to the allocator
    q8t = require_gpu()
    import torch
    calls = _calls(q8t)
    expected = [c() for c in calls]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = calls[0]()
    for n in range(4):
        for t in out:
            t.zero_()
        other = torch.full((1 << (20 + n),), 7, dtype=torch.uint8, device="cuda:0")
        eager = calls[1]()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, expected[0]))
        assert all(torch.equal(x, y) for x, y in zip(eager, expected[1]))
        assert bool((other == 7).all())
        q8t.binding.workspace(q8t.binding.workspace(1, other.device).numel() + (1 << 20), other.device)
