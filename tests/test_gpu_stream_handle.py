"""The stream a call runs on: the current one unless one is given, with or without
torch's getter of its bare handle."""
import pytest

from paper_2410_10447_amd import dock

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("getter", [True, False])
def test_handle_of_the_current_stream(monkeypatch, getter):
    if not getter:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    assert not dock._stream_handle().value                    # the default stream is 0
    with torch.cuda.stream(a):
        assert dock._stream_handle().value == a.cuda_stream
        assert dock._stream_handle(b).value == b.cuda_stream
        with torch.cuda.stream(b):
            assert dock._stream_handle().value == b.cuda_stream
        graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert dock._stream_handle().value == torch.cuda.current_stream().cuda_stream != 0
    assert not dock._stream_handle().value
