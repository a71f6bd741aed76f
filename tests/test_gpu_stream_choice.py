"""The stream a call without one runs on: the calling thread's current stream."""
import threading

import pytest
import torch

import paper_2509_16407_amd as hw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["default", "side", "thread", "given"])
def test_stream_handle(where):
    side = torch.cuda.Stream()
    if where == "default":
        assert hw._stream(None) == torch.cuda.current_stream().cuda_stream
    elif where == "side":
        with torch.cuda.stream(side):
            assert hw._stream(None) == side.cuda_stream
        assert hw._stream(None) != side.cuda_stream
    elif where == "given":
        assert hw._stream(side) == side.cuda_stream
    else:
        got = []
        with torch.cuda.stream(side):  # streams are current per thread
            th = threading.Thread(target=lambda: got.append((hw._stream(None), torch.cuda.current_stream().cuda_stream)))
            th.start()
            th.join()
        assert got[0][0] == got[0][1] != side.cuda_stream
