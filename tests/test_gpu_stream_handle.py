"""The stream handle that calls without a stream pass on: the current device's
current stream, on the null stream, inside a stream context and on threads."""
import threading

import pytest
import torch

from paper_2510_25938_amd import lj

pytestmark = pytest.mark.gpu


def test_handle_is_the_current_streams():
    side = torch.cuda.Stream()
    torch.empty(1, device="cuda")
    assert lj._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert lj._stream() == side.cuda_stream == torch.cuda.current_stream().cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append(
            (lj._stream(), torch.cuda.current_stream().cuda_stream)))
        t.start()
        t.join()
        assert seen[0][0] == seen[0][1]
    assert lj._stream() == torch.cuda.current_stream().cuda_stream
    assert lj._stream(side) == side.cuda_stream
