"""Calls without a stream go to the calling thread's current torch stream."""
import threading

import pytest

from tests.gpu_helpers import torch, vs

pytestmark = pytest.mark.gpu


def test_default_stream_is_the_current_one():
    t, v = torch(), vs()

    def check():
        assert v._stream(None) == t.cuda.current_stream().cuda_stream

    check()
    side = t.cuda.Stream()
    seen = []

    def other():
        check()
        seen.append(v._stream(None))
        with t.cuda.stream(side):
            check()
            seen.append(v._stream(None))

    with t.cuda.stream(side):
        check()
        assert v._stream(None) == side.cuda_stream == v._stream(side) == v._stream(side.cuda_stream)
        th = threading.Thread(target=other)
        th.start()
        th.join()
    check()
    assert seen == [t.cuda.default_stream().cuda_stream, side.cuda_stream]
    g = t.cuda.CUDAGraph()
    x = t.zeros(16, device="cuda")
    with t.cuda.graph(g):
        check()
        x += 1
    check()
