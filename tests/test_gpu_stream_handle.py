"""stream_handle names torch's current stream: the default one, one made
current by a context, nested contexts, and an explicit argument."""
import pytest
import torch

import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu


def test_stream_handle_is_the_current_stream():
    assert fk.stream_handle() == torch.cuda.current_stream().cuda_stream
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        assert fk.stream_handle() == a.cuda_stream
        with torch.cuda.stream(b):
            assert fk.stream_handle() == b.cuda_stream
            assert fk.stream_handle(a) == a.cuda_stream
        assert fk.stream_handle() == a.cuda_stream
    assert fk.stream_handle() == torch.cuda.current_stream().cuda_stream
