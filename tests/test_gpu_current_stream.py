"""The stream handle the binding passes to the library is torch's current stream, on every stream and thread."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_stream_handle_follows_torch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_08368_amd import binding as B
    default = torch.cuda.current_stream().cuda_stream or None
    assert B._stream() == default
    side, seen = torch.cuda.Stream(), []

    def other_thread():
        seen.append(B._stream())

    with torch.cuda.stream(side):
        assert B._stream() == side.cuda_stream
        t = threading.Thread(target=other_thread)
        t.start()
        t.join()
    assert seen == [default] and B._stream() == default
