"""The binding launches on torch's current stream, whichever that is when the call is made."""
import threading

import pytest

from paper_2302_01382_amd import mpq

pytestmark = pytest.mark.gpu


def test_the_current_stream_is_the_one_taken():
    import torch
    assert mpq._stream() == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert mpq._stream() == s.cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append(mpq._stream()))   # a thread has its own current stream
        t.start()
        t.join()
        assert seen == [torch.cuda.default_stream().cuda_stream]
    assert mpq._stream() == torch.cuda.current_stream().cuda_stream
