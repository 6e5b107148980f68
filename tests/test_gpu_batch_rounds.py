"""Residual and image rows of decode batches with several rounds of 32 tokens a workgroup: one token over a round, the last round of one
token, of sixteen and of seventeen, the largest batch, ranks of four steps, eight and sixteen; against 64-bit sums and against calls of fewer tokens."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,ffn,k", [(4096, 16384, 64), (4096, 16384, 256), (2560, 10240, 128), (4096, 12288, 320), (2560, 10240, 96)])
@pytest.mark.parametrize("B", [33, 48, 81, 97, 128])
def test_rounds(d, ffn, k, B):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(d + k + B)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    inputs, maps = [], []
    for i, (n, m) in enumerate([(d, ffn), (ffn, d)]):
        U = torch.linalg.qr(r(n, k)).Q.to(torch.bfloat16).contiguous()
        W = (r(m, n) / n**0.5).to(torch.bfloat16)
        inputs.append({"U": U, "X": r(B, n)})
        maps.append({"W": W, "M": (W.float() @ U.float()).to(torch.bfloat16), "input_id": i})
    print(f"case rounds d={d} ffn={ffn} k={k} B={B}", flush=True)
    st = gsi.LayerStack(inputs, maps, B, 2.0)  # no residual is twice its token: none fires
    st.run()
    torch.cuda.synchronize()
    part = [dict(i, X=i["X"][30:62].contiguous()) for i in inputs]  # (three tokens at least: one takes other kernels)
    n = part[0]["X"].shape[0]
    st2 = gsi.LayerStack(part, maps, n, 2.0)
    st2.run()
    torch.cuda.synchronize()
    for i, (inp, mp) in enumerate(zip(inputs, maps)):
        t = st.inputs_t[i]
        C, x = t["C"].double(), inp["X"].double()
        # of the stored C: 16 mantissa bits of it, 32-bit sums of k products, one subtraction
        bar = lambda b: 2.0**-16 * C.norm(dim=1)[:, None] * b.double().norm(dim=1)[None, :]
        assert ((st.maps_t[i]["Y"].double() - C @ mp["M"].double().T).abs() <= bar(mp["M"])).all()
        assert ((t["R"].double() - (x - C @ inp["U"].double().T)).abs() <= bar(inp["U"]) + 2.0**-23 * x.abs()).all()
        assert ((t["rnorm"].double() - t["R"].double().norm(dim=1)).abs() <= 2.0**-20 * t["R"].double().norm(dim=1)).all()
        assert int(t["n_fired"][0]) == 0
        # a token's coefficients, residual and image term are the same whatever its batch
        for key in ("C", "R"):
            assert torch.equal(st2.inputs_t[i][key], t[key][30:30 + n]), key
        assert torch.equal(st2.maps_t[i]["Y"], st.maps_t[i]["Y"][30:30 + n])
