"""The binding takes the raw handle of the current stream without a Stream
object; it is the handle of torch's public interface, on every stream, and work
goes to that stream."""
import numpy as np
import pytest

from paper_0912_0180_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_handle_is_the_current_streams():
    import torch
    from paper_0912_0180_amd import hh
    t = torch.zeros(1, device="cuda")
    assert hh._stream(t) == torch.cuda.current_stream(t.device).cuda_stream
    seen = set()
    for _ in range(3):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            assert hh._stream(t) == s.cuda_stream != 0
            seen.add(hh._stream(t))
    assert len(seen) == 3


def test_calls_run_on_the_current_stream():
    import torch
    from paper_0912_0180_amd import hh
    c = W.c1()
    g = hh.Grid(c["desc"], c["phi"])
    b = torch.from_numpy(c["b"]).cuda()
    want, cyc = g.apply(b).clone(), g.vcycle(b).clone()
    f, y, u = torch.zeros_like(b), torch.empty_like(b), torch.empty_like(b)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        torch.cuda._sleep(20000000)      # f is written late on this stream
        f.copy_(b)
        g.apply(f, out=y)
        g.vcycle(f, out=u)
    s.synchronize()
    assert torch.equal(y, want) and torch.equal(u, cyc)
