"""The binding's default stream is torch's current stream, in every context and thread."""
import threading

import pytest
import torch

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
abi = mx.abi


def test_default_stream_is_torchs_current_stream():
    def check():
        assert abi._stream(None) == torch.cuda.current_stream().cuda_stream

    check()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        check()
        assert abi._stream(None) == a.cuda_stream
        with torch.cuda.stream(b):
            check()
        check()
        seen = []
        t = threading.Thread(target=lambda: seen.append(abi._stream(None)))  # a thread has a current stream of its own
        t.start()
        t.join()
        assert seen == [torch.cuda.default_stream().cuda_stream]
    check()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        check()
    assert abi._stream(b) == b.cuda_stream and abi._stream(7) == 7
