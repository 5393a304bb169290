"""The stream that a call without one goes to is torch's current one of the current device, call by call and thread by thread."""
import threading

import pytest

from paper_2602_06694_amd import binding as nq

pytestmark = pytest.mark.gpu


def test_current_stream_is_followed():
    import torch
    want = lambda: torch.cuda.current_stream().cuda_stream or None
    assert nq._stream(None) == want() and nq._stream(None) == want()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    seen = []
    with torch.cuda.stream(a):
        assert nq._stream(None) == want() == a.cuda_stream
        with torch.cuda.stream(b):
            assert nq._stream(None) == want() == b.cuda_stream
            t = threading.Thread(target=lambda: seen.append((nq._stream(None), want())))       # a thread has its own current stream
            t.start()
            t.join()
        assert nq._stream(None) == a.cuda_stream
    assert seen[0][0] == seen[0][1] != b.cuda_stream
    assert nq._stream(None) == want()
    assert nq._stream(a) == a.cuda_stream and nq._stream(0) is None
    nq._forget_raw_stream()
    assert nq._stream(None) == want()


def test_capture_goes_to_the_captured_stream():
    import torch
    x = torch.arange(64, dtype=torch.float32, device="cuda").reshape(1, 64)
    out = torch.zeros(64, device="cuda")
    nq.nq_scale_grad(x, nq.NQ_F32, x, nq.NQ_F32, 1, 64, out)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        nq.nq_scale_grad(x, nq.NQ_F32, x, nq.NQ_F32, 1, 64, out)
    for k in range(3):
        x.fill_(float(k + 2))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, torch.full_like(out, float(k + 2) ** 2))
