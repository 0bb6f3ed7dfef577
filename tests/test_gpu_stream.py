"""torch_glue hands the C ABI the stream that torch has current: the default one, another one, and after leaving it."""
import pytest

torch = pytest.importorskip("torch")

from paper_2506_13472_amd import torch_glue as T

pytestmark = pytest.mark.gpu


def test_current_stream_pointer():
    print("case current stream", flush=True)
    torch.zeros(1, device="cuda")
    assert T.current_stream_ptr() == torch.cuda.current_stream().cuda_stream
    streams = [torch.cuda.Stream() for _ in range(3)]
    for s in streams:
        with torch.cuda.stream(s):
            assert T.current_stream_ptr() == s.cuda_stream
    assert len({s.cuda_stream for s in streams}) == 3
    assert T.current_stream_ptr() == torch.cuda.default_stream().cuda_stream
