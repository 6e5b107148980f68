"""The binding's own scratch buffers: never shared by calls that may overlap, bounded, and not kept from a capture."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_a_buffer_per_stream_and_thread():
    from paper_2605_03109_amd import gsi

    here = gsi.workspace(1000)
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(s):
        on_s = gsi.workspace(1000)
    assert here.data_ptr() != on_s.data_ptr()
    assert len({here.data_ptr(), on_s.data_ptr(), gsi.workspace(1000, stream=t).data_ptr()}) == 3
    assert gsi.workspace(1000).data_ptr() == here.data_ptr() and gsi.workspace(1000, stream=s).data_ptr() == on_s.data_ptr()
    other = []
    th = threading.Thread(target=lambda: other.append(gsi.workspace(1000)))
    th.start()
    th.join()
    assert other[0].data_ptr() != here.data_ptr()
    assert gsi.workspace(3 << 20).numel() >= 3 << 20 and gsi.workspace(0) is None


def test_buffers_are_bounded():
    from paper_2605_03109_amd import gsi

    streams = [torch.cuda.Stream() for _ in range(12)]
    for st in streams:
        gsi.workspace(1000, stream=st)
    assert len(gsi._ws_local.__dict__) <= gsi._WS_KEPT


def test_captured_call_uses_the_graphs_memory():
    """A graph replayed beside eager calls that outgrow the kept buffer: both stay right."""
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(1)
    d, k, T = 1024, 64, 20
    U = torch.linalg.qr(torch.randn(d, k, generator=g, device="cuda"))[0].to(torch.bfloat16).contiguous()
    X = torch.randn(T, d, generator=g, device="cuda")
    want = [o.clone() for o in gsi.project(U, X)]
    out = [torch.empty_like(o) for o in want]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gsi.project(U, X, *out)
    grown = torch.randn(128, 4096, generator=g, device="cuda")
    Ug = torch.linalg.qr(torch.randn(4096, 256, generator=g, device="cuda"))[0].to(torch.bfloat16).contiguous()
    for _ in range(3):
        for o in out:
            o.fill_(float("nan"))
        gsi.project(Ug, grown)
        graph.replay()
        gsi.project(Ug, grown)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(want, out))
