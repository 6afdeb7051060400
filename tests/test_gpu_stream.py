"""Calls without a stream argument run on the calling thread's current stream."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_current_stream_of_the_calling_thread():
    import torch
    import paper_2108_01438_amd as P
    assert P._stream_ptr() == torch.cuda.current_stream().cuda_stream
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    seen = {}

    def other():
        seen["default"] = P._stream_ptr()
        with torch.cuda.stream(b):
            seen["b"] = P._stream_ptr()

    with torch.cuda.stream(a):
        t = threading.Thread(target=other)
        t.start()
        t.join()
        assert P._stream_ptr() == a.cuda_stream
        assert P._stream_ptr(b) == b.cuda_stream
    assert seen == {"default": torch.cuda.default_stream().cuda_stream, "b": b.cuda_stream}
    assert P._stream_ptr() == torch.cuda.current_stream().cuda_stream
