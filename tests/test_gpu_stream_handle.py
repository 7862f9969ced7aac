"""The binding's handle of the current stream, with and without torch's raw call."""

import pytest
import torch

import paper_1105_2279_amd as q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream_handle(raw, monkeypatch):
    if not raw:
        monkeypatch.setattr(q, "_raw_stream", None)
    assert q._stream() == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert q._stream() == s.cuda_stream
    assert q._stream(s) == s.cuda_stream and q._stream(5) == 5
