"""One token, step by step: the calls of their own against the whole call, bit for bit, and replayed from a graph."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# fewer rows than waves; one row per wave and some with two; several; a rank of one piece, ragged and of 64 pieces;
# whole units of columns and tails; columns taken in blocks
@pytest.mark.parametrize("d,k,m,dtype", [
    (1024, 8, 1, "bf16"), (768, 64, 3072, "f32"), (4096, 256, 8200, "bf16"), (1160, 200, 264, "bf16"), (1024, 512, 20000, "bf16"),
    (1160, 136, 7, "f32"), (2048, 256, 16390, "f32"), (20480, 64, 300, "bf16"), (4096, 24, 4099, "bf16"), (2176, 4, 5000, "f32")])
@pytest.mark.parametrize("eps", [1e-3, 10.0])  # the token fires / does not
def test_calls_of_one_token(d, k, m, dtype, eps):
    from paper_2605_03109_amd import gsi

    print(f"case one token d={d} k={k} m={m} {dtype} eps={eps}", flush=True)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator(device="cuda").manual_seed(d + k + m)
    U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).to(dt)
    W = (torch.randn(m, d, generator=g, device="cuda") / d**0.5).to(dt)
    M = (W.double() @ U.double()).to(dt)
    X = torch.randn(1, d, generator=g, device="cuda")
    st = gsi.layer_stack([{"U": U, "X": X}], [{"W": W, "M": M, "input_id": 0}], 1, eps)
    f32 = dict(device="cuda", dtype=torch.float32)
    C, R, rn, xn, Y = [torch.zeros(s, **f32) for s in ((1, k), (1, d), (1,), (1,), (1, m))]
    mask = torch.zeros(1, device="cuda", dtype=torch.uint8)
    idx, nf = [torch.zeros(1, device="cuda", dtype=torch.int32) for _ in range(2)]
    ws = torch.empty(max(gsi.workspace_bytes(c, m, d, k, 1) for c in (gsi.CALL_PROJECT, gsi.CALL_GATED_LINEAR)),
                     device="cuda", dtype=torch.uint8).fill_(255)

    def calls():
        gsi.project(U, X, C, R, rn, xn, ws=ws)
        gsi.gate(rn, xn, eps, mask, idx, nf)
        gsi.gated_linear(W, M, C, R, idx, nf, Y, ws=ws)

    def check():
        torch.cuda.synchronize()
        t = st.inputs_t[0]
        for a, b in ((C, t["C"]), (R, t["R"]), (rn, t["rnorm"]), (xn, t["xnorm"]), (mask, t["mask"]), (nf, t["n_fired"])):
            assert torch.equal(a, b)
        assert torch.equal(Y, st.maps_t[0]["Y"])

    calls()
    check()
    assert int(nf) == (1 if eps < 1 else 0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    for _ in range(3):
        for t in (C, R, rn, xn, Y):
            t.fill_(7.0)
        graph.replay()
        check()
        calls()  # eager work between the replays
        check()
