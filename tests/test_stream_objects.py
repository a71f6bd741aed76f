"""Streams as a caller may hand them over: any object with the stream's handle (CPU only)."""
import torch

import paper_2509_16407_amd as hw


class Handle:
    cuda_stream = 4096


def test_an_object_with_a_handle_alone_runs_the_plain_call():
    """Its device is not known, so no scratch memory is taken for it."""
    assert hw._stream(Handle()) == 4096
    assert hw._scratch_memory(1 << 20, torch.device("cuda", 0), Handle()) is None
