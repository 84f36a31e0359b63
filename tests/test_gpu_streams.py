"""The stream a call without one is given: the calling thread's current stream,
looked up per call."""
import threading

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2410_05934_amd as ntt  # noqa: E402


def test_default_stream_argument_follows_the_current_stream_of_the_thread():
    side = torch.cuda.Stream()
    home = torch.cuda.current_stream().cuda_stream
    assert ntt._stream_handle(None) == home
    seen = []
    with torch.cuda.stream(side):
        assert ntt._stream_handle(None) == side.cuda_stream != home
        worker = threading.Thread(target=lambda: seen.append(ntt._stream_handle(None)))
        worker.start()
        worker.join()
    assert seen == [torch.cuda.default_stream().cuda_stream]
    assert ntt._stream_handle(None) == home
    assert ntt._stream_handle(side) == side.cuda_stream
