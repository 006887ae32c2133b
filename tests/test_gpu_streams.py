"""Calls without a stream go to the stream that is current when they are made."""
import pytest

pytestmark = pytest.mark.gpu


def test_default_stream_argument_is_the_current_stream():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_00662_amd as m
    side = torch.cuda.Stream()
    src = torch.arange(1 << 20, dtype=torch.int32, device="cuda")
    for stream in (torch.cuda.current_stream(), side, torch.cuda.current_stream()):
        with torch.cuda.stream(stream):
            assert m.binding._stream(None) == torch.cuda.current_stream().cuda_stream == stream.cuda_stream
            dst = torch.zeros_like(src)
            stream.synchronize()
            m.monta_copy(dst, src, src.numel() * 4)
            stream.synchronize()
            assert torch.equal(dst, src)


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_the_undocumented_functions(monkeypatch, missing):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_00662_amd as m
    side = torch.cuda.Stream()          # also initialises torch's side, which uses the functions itself
    monkeypatch.setattr(m.binding, "_raw_stream", None)
    with torch.cuda.stream(side):
        want = torch.cuda.current_stream().cuda_stream
        monkeypatch.delattr(torch._C, missing)
        monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: side)
        assert m.binding._stream(None) == want == side.cuda_stream
        monkeypatch.undo()
