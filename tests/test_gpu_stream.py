"""Calls without a stream argument run on torch's current stream of the current
device: the default stream, a side stream, nested, inside a capture, and per
thread."""
from __future__ import annotations

import threading

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2601_03324_amd import tvl  # noqa: E402


def same():
    return tvl._stream(None) == torch.cuda.current_stream().cuda_stream


def test_current_stream_handle():
    torch.zeros(1, device="cuda")
    assert same()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        assert same() and tvl._stream(None) == a.cuda_stream
        with torch.cuda.stream(b):
            assert same() and tvl._stream(None) == b.cuda_stream
        seen = []  # a new thread starts on the default stream
        t = threading.Thread(target=lambda: seen.append((tvl._stream(None), same())))
        t.start()
        t.join()
        assert seen == [(torch.cuda.default_stream().cuda_stream, True)]
        assert tvl._stream(None) == a.cuda_stream
    assert tvl._stream(None) == torch.cuda.default_stream().cuda_stream
    assert tvl._stream(b) == b.cuda_stream and tvl._stream(7) == 7


def test_capture_uses_the_capturing_stream():
    M = K = 256
    W, x = torch.ones(M, K, device="cuda"), torch.ones(K, device="cuda")
    y = torch.zeros(M, device="cuda")
    tvl.tvl_gemv(W, K, tvl.TVL_F32, x, y, M, K)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        assert same()
        tvl.tvl_gemv(W, K, tvl.TVL_F32, x, y, M, K)
    for v in (2.0, 3.0, 4.0):
        x.fill_(v)
        g.replay()
        torch.cuda.synchronize()
        assert bool((y == v * K).all())
