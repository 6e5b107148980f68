"""Residual rows and image terms of calls of many more tiles than the chip holds: a workgroup takes tile after tile, from a product of one rank
to one of another, and requests the operands of the next beside the last products of the one before."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# (512 workgroups; 900 tiles through the caches, 3000 past them) ranks of two, six and sixteen k-tiles; rows and columns with remainders
@pytest.mark.parametrize("xdtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B", [1490, 5001])
def test_ranks_in_turn(B, xdtype):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(B)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    shapes = [(2048, 64, (8192, 36)), (1088, 192, (2308,)), (4096, 512, (1000,)), (320, 128, ())]
    inputs, maps = [], []
    for i, (d, k, ms) in enumerate(shapes):
        U = torch.linalg.qr(r(d, k)).Q.to(torch.bfloat16).contiguous()
        inputs.append({"U": U, "X": r(B, d).to(xdtype)})
        for m in ms:
            W = (r(m, d) / d**0.5).to(torch.bfloat16)
            maps.append({"W": W, "M": (W.float() @ U.float()).to(torch.bfloat16), "input_id": i})
    print(f"case ranks in turn B={B} x {xdtype}", flush=True)
    st = gsi.LayerStack(inputs, maps, B, 2.0)  # no residual is twice its token: none fires
    st.run()
    for t in st.inputs_t:
        out = gsi.project(t["U"], t["X"])
        torch.cuda.synchronize()
        for got, key in zip(out, ("C", "R", "rnorm", "xnorm")):
            assert torch.equal(got, t[key]), key
        C, x, U = t["C"].double(), t["X"].double(), t["U"].double()
        # of the stored C: 16 mantissa bits of it, 32-bit sums of k products, one subtraction; norms of the stored rows, 32-bit sums of d squares
        assert ((t["R"].double() - (x - C @ U.T)).abs() <= 2.0**-16 * C.norm(dim=1)[:, None] * U.norm(dim=1)[None, :] + 2.0**-23 * x.abs()).all()
        for got, rows in ((t["rnorm"], t["R"].double()), (t["xnorm"], x)):
            assert ((got.double() - rows.norm(dim=1)).abs() <= 2.0**-20 * rows.norm(dim=1)).all()
        assert int(t["n_fired"][0]) == 0
    for mt in st.maps_t:
        t = st.inputs_t[mt["input_id"]]
        y = gsi.gated_linear(mt["W"], mt["M"], t["C"], t["R"], t["fired_idx"], t["n_fired"])
        torch.cuda.synchronize()
        assert torch.equal(y, mt["Y"])
        C, M = t["C"].double(), mt["M"].double()
        assert ((mt["Y"].double() - C @ M.T).abs() <= 2.0**-16 * C.norm(dim=1)[:, None] * M.norm(dim=1)[None, :]).all()
