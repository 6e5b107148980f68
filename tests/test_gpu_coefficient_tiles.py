"""Coefficients of bf16 tokens, whose tiles are of 64 rows in a launch that leaves half the chip idle and of 128 in a larger one: a projection has
the same bits by itself and beside others, and those of its 64-bit sums to rounding."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# rows and columns with remainders, one k-tile, an odd number; unsplit, in parts; the last and the first number of inputs (of 128 workgroups in all, and more)
@pytest.mark.parametrize("d,k,B,n", [(64, 64, 1001, 24), (192, 192, 800, 24), (1088, 320, 257, 24), (2048, 256, 640, 16), (4096, 512, 2049, 4), (1024, 64, 500, 8),
                                     (1024, 64, 500, 9)])
def test_alone_and_beside(d, k, B, n):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(d + k + B)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    U = (r(d, k) / d**0.5).to(torch.bfloat16)
    W = (r(8, d) / d**0.5).to(torch.bfloat16)
    M = (W.float() @ U.float()).to(torch.bfloat16)
    X = [r(B, d).to(torch.bfloat16) for _ in range(n)]
    print(f"case coefficient tiles d={d} k={k} B={B} inputs={n}", flush=True)
    st = gsi.LayerStack([{"U": U, "X": x} for x in X], [{"W": W, "M": M, "input_id": i} for i in range(n)], B, 10.0)
    st.run()
    for i in (0, n // 2, n - 1):
        out = gsi.project(U, X[i])
        torch.cuda.synchronize()
        for got, key in zip(out, ("C", "R", "rnorm", "xnorm")):
            assert torch.equal(got, st.inputs_t[i][key]), key
        x, u = X[i].double(), U.double()
        # 32-bit sums of d exact products
        assert ((out[0].double() - x @ u).abs() <= (8 + d**0.5) * 2.0**-24 * (x.abs() @ u.abs())).all()
