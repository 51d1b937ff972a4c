"""Calls without a stream argument run on torch's current stream: the default
one, one entered as a context, and a capturing one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2403_01876_amd import dv  # noqa: E402


def test_current_stream_is_used():
    assert dv._stream(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert dv._stream(None) == side.cuda_stream
    assert dv._stream(None) == torch.cuda.current_stream().cuda_stream != side.cuda_stream
    x = torch.arange(2 * 2 * 3 * 16 * 64, dtype=torch.int16, device="cuda")
    c = dv.Cache(dv.DV_DENSE, 1, 3, 64, 4, [x], max_seq=8)
    pos = np.array([1, 0, 7, 3], np.int32)
    wire = torch.zeros(dv.dv_packed_bytes(c, 0, 1, pos, pos + 1), dtype=torch.uint8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):  # a call on another stream would not be captured
        dv.dv_stream_out_token(c, 0, 0, 1, pos, wire, wire.numel())
    torch.cuda.synchronize()
    assert not bool(wire.any())
    want = x.view(2, 4, 3, 8, 64)[:, torch.arange(4), :, torch.from_numpy(pos).long()]
    for _ in range(3):
        wire.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(wire.view(torch.int16), want.permute(1, 0, 2, 3).reshape(-1))
