"""The scratch memory behind the Python calls: one buffer per stream, none shared with a captured graph."""
import pytest
import torch


@pytest.fixture
def ws(monkeypatch):
    # the bookkeeping alone, on CPU memory: the stream and the capture state come from the test
    from paper_1805_11046_amd import binding
    state = {"stream": 1, "capturing": False}
    monkeypatch.setattr(binding, "_stream", lambda: state["stream"])
    monkeypatch.setattr(binding, "_capturing", lambda: state["capturing"], raising=False)
    monkeypatch.setattr(binding, "_ws_cache", {})
    state["get"] = lambda n: binding.workspace(n, torch.device("cpu"))
    state["cache"] = binding._ws_cache
    return state


def test_streams_do_not_share_a_buffer(ws):
    a = ws["get"](1000)
    assert ws["get"](500) is a
    ws["stream"] = 2
    b = ws["get"](1000)
    assert b.data_ptr() != a.data_ptr()
    grown = ws["get"](5000)
    assert grown.numel() >= 5000 and ws["get"](10) is grown
    ws["stream"] = 1
    assert ws["get"](1000) is a


def test_number_of_buffers_is_bounded(ws):
    for i in range(100):
        ws["stream"] = i
        ws["get"](300)
    assert len(ws["cache"]) <= 16
    assert ws["get"](300) is ws["get"](300)


def test_captured_calls_keep_no_buffer(ws):
    a = ws["get"](1000)
    ws["capturing"] = True
    b, c = ws["get"](1000), ws["get"](1000)
    assert len({a.data_ptr(), b.data_ptr(), c.data_ptr()}) == 3
    ws["capturing"] = False
    assert ws["get"](1000) is a
