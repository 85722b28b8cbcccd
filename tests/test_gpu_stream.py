"""Calls without a stream argument go to torch's current stream: of the calling thread, inside `with torch.cuda.stream`, under
graph capture."""
import threading

import pytest

import paper_2110_15032_amd as sbp
from paper_2110_15032_amd.binding import _stream_ptr

pytestmark = pytest.mark.gpu


def test_current_stream():
    import torch

    def same():
        return (_stream_ptr(None).value or 0) == torch.cuda.current_stream().cuda_stream

    assert same()
    side = torch.cuda.Stream()
    seen = []
    with torch.cuda.stream(side):
        assert same() and _stream_ptr(None).value == side.cuda_stream
        t = threading.Thread(target=lambda: seen.append((same(), (_stream_ptr(None).value or 0) != side.cuda_stream)))
        t.start()
        t.join()
    assert same() and seen == [(True, True)]

    src = torch.arange(64, dtype=torch.float32, device="cuda")
    out = [torch.zeros(64, device="cuda") for _ in range(2)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert same()
        sbp.sbp_boxing(sbp.SbpTensor([src, src], 8, 8, sbp.F32), sbp.P_SUM, sbp.SbpTensor(out, 8, 8, sbp.F32), sbp.B, 2)
    for i in range(1, 4):
        src.fill_(i)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o, torch.full_like(o, 2.0 * i)) for o in out)
