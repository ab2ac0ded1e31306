"""What decode_step refuses, and with which error; and that it launches on
torch's current stream (a side stream, eager and captured)."""
import pytest

from tests.ssd_harness import announce
from tests.test_gpu_parity import _gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def operands(dtype):
    import torch

    g = torch.Generator().manual_seed(5)
    n = lambda *s: torch.randn(s, generator=g).cuda()
    return dict(x=n(2, 4, 64).to(dtype), dt=n(2, 4).abs().to(dtype), A_log=n(4), B=n(2, 1, 128).to(dtype),
                C=n(2, 1, 128).to(dtype), state=n(2, 4, 64, 128), D=n(4))


@pytest.mark.parametrize("name,change,error", [
    ("x", lambda t: t.half(), TypeError), ("x", lambda t: t.cpu(), ValueError),
    ("dt", lambda t: t.float(), TypeError), ("B", lambda t: t.float(), TypeError), ("C", lambda t: t.float(), TypeError),
    ("A_log", lambda t: t.double(), TypeError), ("state", lambda t: t.bfloat16(), TypeError),
    ("D", lambda t: t.bfloat16(), TypeError), ("D", lambda t: t.cpu(), ValueError), ("C", lambda t: t.cpu(), ValueError),
    ("x", lambda t: t.transpose(0, 1).contiguous().transpose(0, 1), ValueError),
    ("state", lambda t: t.transpose(2, 3).contiguous().transpose(2, 3), ValueError),
    ("A_log", lambda t: None, RuntimeError), ("state", lambda t: None, RuntimeError),
])
def test_refusals(name, change, error):
    import torch
    from paper_2405_21060_amd import ssd

    announce("decode refuses %s" % name)
    o = operands(torch.bfloat16)
    o[name] = change(o[name])
    with pytest.raises(error):
        ssd.decode_step(**o)


def test_streams():
    import torch
    from paper_2405_21060_amd import ssd

    announce("decode on a side stream and captured")
    o = operands(torch.bfloat16)
    start = o["state"].clone()
    y0 = ssd.decode_step(**o)
    s0 = o["state"].clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    o["state"].copy_(start)
    with torch.cuda.stream(side):
        side.wait_stream(torch.cuda.default_stream())
        y1 = ssd.decode_step(**o)
    side.synchronize()
    assert torch.equal(y0, y1) and torch.equal(s0, o["state"])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y2 = ssd.decode_step(**o)
    for _ in range(3):
        o["state"].copy_(start)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y0, y2) and torch.equal(s0, o["state"])
