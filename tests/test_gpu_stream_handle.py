"""The binding launches on torch's current stream, whichever that is."""
import pytest

torch = pytest.importorskip("torch")

import paper_1505_05655_amd as rc  # noqa: E402

pytestmark = pytest.mark.gpu


def test_calls_go_to_the_current_stream():
    assert rc._stream(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert rc._stream(None) == side.cuda_stream
    assert rc._stream(None) == torch.cuda.current_stream().cuda_stream
    assert rc._stream(side) == side.cuda_stream and rc._stream(7) == 7
