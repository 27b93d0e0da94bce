"""A call without a stream runs on the caller's current stream, whichever that
is: the handle follows a stream context, its end, and another thread's own."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_handle_follows_the_current_stream():
    from paper_2511_19457_amd import abi
    torch.zeros(1, device="cuda")
    default = torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    assert abi._stream(None) == default
    seen = []
    with torch.cuda.stream(side):
        assert abi._stream(None) == side.cuda_stream
        t = threading.Thread(target=lambda: seen.append(abi._stream(None)))
        t.start()
        t.join()
    assert abi._stream(None) == default and seen == [default]
    assert abi._stream(side) == abi._stream(side.cuda_stream) == side.cuda_stream
