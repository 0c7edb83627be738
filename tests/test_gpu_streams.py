"""Calls without a stream argument run on the calling thread's current stream
of the current device."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_default_stream_is_the_current_one():
    import torch
    from paper_2507_00528_amd import nep
    side = torch.cuda.Stream()
    seen = []

    def look():
        seen.append((nep._stream(), torch.cuda.current_stream().cuda_stream))

    look()
    with torch.cuda.stream(side):
        look()
        other = threading.Thread(target=look)   # a new thread is on the default stream
        other.start()
        other.join()
    look()
    assert all(a == b for a, b in seen)
    assert seen[1][0] == side.cuda_stream != seen[0][0] == seen[2][0] == seen[3][0]
    assert nep._stream(side) == side.cuda_stream
