"""gsi_gated_linear of more than 128 tokens by itself: its image term from c as it is in memory, against 64-bit sums and, bit for bit,
against the stack, whose image terms share a launch; and the launches of a call."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


# row tiles of 64 and column tiles of 256 with remainders; two k-tiles, an odd number of pairs of them; as many tiles as two and three a unit
# hold, and one row of tiles more, at the last rank that is split on its way whatever the tiles, and the next
@pytest.mark.parametrize("m,d,k,B", [(4, 64, 64, 129), (260, 192, 192, 191), (1028, 320, 320, 257), (16384, 192, 192, 512), (16384, 192, 192, 513),
                                     (16380, 256, 256, 768), (16384, 256, 256, 769), (16384, 192, 192, 769), (36, 512, 512, 1000)])
def test_image_term(m, d, k, B):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(m + d + k + B)
    U = torch.linalg.qr(torch.randn(d, k, generator=g, device="cuda").double()).Q.to(torch.bfloat16).contiguous()
    X = torch.randn(B, d, generator=g, device="cuda")
    W = (torch.randn(m, d, generator=g, device="cuda") / d**0.5).to(torch.bfloat16)
    M = (W.double() @ U.double()).to(torch.bfloat16)
    M[1, 0], M[2, :] = float("inf"), float("nan")  # stay in their columns of Y
    print(f"case image term m={m} d={d} k={k} B={B}", flush=True)
    st = gsi.LayerStack([{"U": U, "X": X}], [{"W": W, "M": M, "input_id": 0}], B, 2.0)  # no residual is twice its token: none fires
    st.run()
    t = st.inputs_t[0]
    Y = torch.full((B + 1, m), 7.0, device="cuda")
    gsi.gated_linear(W, M, t["C"], t["R"], t["fired_idx"], t["n_fired"], Y=Y[:B])
    torch.cuda.synchronize()
    assert torch.equal(Y[:B].view(torch.int32), st.maps_t[0]["Y"].view(torch.int32)) and bool((Y[B] == 7.0).all())
    rest = [j for j in range(m) if j not in (1, 2)]
    C, N = t["C"].double(), M.double()
    # of the stored C: 16 mantissa bits of it, 32-bit sums of k products
    bar = 2.0**-16 * C.norm(dim=1)[:, None] * N.norm(dim=1)[None, :]
    assert ((Y[:B].double() - C @ N.T).abs() <= bar)[:, rest].all()
    assert not Y[:B, 1].isfinite().any() and Y[:B, 2].isnan().all()


# the image term, the W term and the sums of its parts: c and the fired rows take no launch of their own
@pytest.mark.parametrize("m,d,k,B", [(1024, 1024, 64, 300), (2048, 2048, 128, 1100)])
def test_launches(m, d, k, B):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(m + d + k + B)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    W, M, C, R = (r(m, d) / d**0.5).to(torch.bfloat16), (r(m, k) / k**0.5).to(torch.bfloat16), r(B, k), r(B, d)
    idx, count = torch.arange(B, dtype=torch.int32, device="cuda"), torch.tensor([B // 5], dtype=torch.int32, device="cuda")
    Y = torch.empty(B, m, device="cuda")
    ws = torch.empty(gsi.workspace_bytes(gsi.CALL_GATED_LINEAR, m, d, k, B), dtype=torch.uint8, device="cuda")
    print(f"case launches m={m} d={d} k={k} B={B}", flush=True)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        gsi.gated_linear(W, M, C, R, idx, count, Y=Y, ws=ws)
    n = ctypes.c_size_t(0)
    nodes = gsi.lib.hipGraphGetNodes
    nodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    assert nodes(graph.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    assert n.value == 3
    graph.instantiate()
    want = gsi.gated_linear(W, M, C, R, idx, count).clone()
    for _ in range(3):
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
