"""The stream that a call without one runs on: torch's current stream, also where torch has no private read of it."""
import pytest

from gpu_helpers import gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("private", [True, False])
def test_current_stream(monkeypatch, private):
    gpu()
    from paper_2204_03139_amd import _lib
    if not private:
        monkeypatch.setattr(_lib, "_raw_stream", None)
    side = torch.cuda.Stream()
    assert _lib._stream() == torch.cuda.current_stream().cuda_stream
    assert _lib._stream(side) == side.cuda_stream
    with torch.cuda.stream(side):
        assert _lib._stream() == side.cuda_stream
