"""Image terms that ride in the residual launch of a bf16 decode batch: one and several rounds of 32 tokens, row counts
that are no multiple of 128, ranks of two and of three operand terms, whole slices and remainders.

The bars are those of parity_util against the fp64 oracle; a map whose Y lies over an x of the call keeps its image in
the launch of the weight term, and a stack equals separate calls bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _make(d, ms, k, B, xdtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    U = torch.linalg.qr(n(d, k).double())[0].to(torch.bfloat16).contiguous()
    X = (n(B, k) @ U.float().T + 0.2 * n(B, 1).abs() * n(B, d) / d**0.5).to(xdtype)
    Ws = [(n(m, d) / d**0.5).to(torch.bfloat16) for m in ms]
    return U, X, Ws, [(W.float() @ U.float()).to(torch.bfloat16) for W in Ws]


def _stack(gsi, U, X, Ws, Ms, B, flags=0, ys=None):
    maps = [{"W": W, "M": M, "input_id": 0} for W, M in zip(Ws, Ms)]
    for mp, y in zip(maps, ys or []):
        if y is not None:
            mp["Y"] = y
    return gsi.layer_stack([{"U": U, "X": X, "flags": flags}], maps, B, 0.15)


@pytest.mark.parametrize("wx", [False, True])
@pytest.mark.parametrize("k,xdtype", [(64, torch.float32), (256, torch.bfloat16), (200, torch.float32), (512, torch.float32)])
@pytest.mark.parametrize("B", [2, 16, 17, 32, 33, 100, 128])
def test_images_beside_residuals(B, k, xdtype, wx):
    from paper_2605_03109_amd import gsi

    d, ms = 1024, [1024, 132, 516]
    U, X, Ws, Ms = _make(d, ms, k, B, xdtype, 7 * B + k)
    st = _stack(gsi, U, X, Ws, Ms, B, gsi.INPUT_SLOW_PATH_WX if wx else 0)
    t = st.inputs_t[0]
    x, u = X.double(), U.double()
    c = x @ u
    # c: d products of values below |x|: sqrt(d) roundings of 2^-24 of the norm, with a factor 8 for the worst entry
    assert (t["C"].double() - c).abs().max() <= 8 * d**0.5 * 2.0**-24 * x.norm(dim=1).max()
    nf = int(t["n_fired"].item())
    fired = t["fired_idx"][:nf].long()
    for W, M, mp in zip(Ws, Ms, st.maps_t):
        y = c @ M.double().T
        if nf:
            full = x[fired] @ W.double().T
            y[fired] = full if wx else y[fired] + t["R"][fired].double() @ W.double().T
        # operands split into two bf16 terms keep 2^-17 of each value; the sum of d of them: the norm of the vector
        # times the norm of the row of weights, which bounds every |y|
        bar = 2.0**-16 * (c.norm(dim=1).max() * M.double().norm(dim=1).max() + x.norm(dim=1).max() * W.double().norm(dim=1).max())
        assert (mp["Y"].double() - y).abs().max() <= bar
    # separate calls take the image beside the weight term: the same products in the same order
    if not wx:
        for W, M, mp in zip(Ws, Ms, st.maps_t):
            y = gsi.gated_linear(W, M, t["C"], t["R"], t["fired_idx"], t["n_fired"])
            assert torch.equal(y, mp["Y"])


def test_output_over_an_input():
    """Y of the second map is the buffer that X of the same call lies in (m = d, fp32): x is read before it is written."""
    from paper_2605_03109_amd import gsi

    d, B, k = 1024, 40, 64
    U, X, Ws, Ms = _make(d, [512, d], k, B, torch.float32, 3)
    want = _stack(gsi, U, X.clone(), Ws, Ms, B)
    have = _stack(gsi, U, X, Ws, Ms, B, ys=[None, X])
    assert want.maps_t[0]["Y"].abs().max() > 0
    for a, b in zip(want.maps_t, have.maps_t):
        assert torch.equal(a["Y"], b["Y"])
    for n in ("C", "R", "rnorm", "xnorm", "mask", "n_fired"):
        assert torch.equal(want.inputs_t[0][n], have.inputs_t[0][n])
