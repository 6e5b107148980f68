"""Decode batches whose fp32 operand enters as three bf16 terms: an infinite weight gives the infinity of the fp32 product,
not the NaN of an infinity times a remainder; everything else keeps its bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _same_infinities(got, value):
    """got is +inf where value > 0, -inf where value < 0."""
    assert (value != 0).all() and torch.equal(got, torch.sign(value) * float("inf")), got


@pytest.mark.parametrize("T", [5, 40, 100])
def test_one_infinite_weight(T):
    from paper_2605_03109_amd import gsi

    d, k, m = 1024, 200, 260
    g = torch.Generator(device="cuda").manual_seed(T)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    U = torch.linalg.qr(r(d, k).double())[0].to(torch.bfloat16).contiguous()
    X, Xb = r(T, d), r(T, d).to(torch.bfloat16)  # the residual is most of x: every token fires
    W = (r(m, d) / d**0.5).to(torch.bfloat16)
    M = (W.float() @ U.float()).to(torch.bfloat16)
    Wi, Mi, Ui = W.clone(), M.clone(), U.clone()
    Wi[5, 7] = Mi[9, 3] = Ui[17, 11] = float("inf")
    rest = [i for i in range(m) if i not in (5, 9)]
    stack = lambda W, M, x, flags: gsi.layer_stack([{"U": U, "X": x, "flags": flags}], [{"W": W, "M": M, "input_id": 0}], T, 0.05)
    for x, flags in ((X, 0), (Xb, 0), (Xb, gsi.INPUT_SLOW_PATH_WX)):
        clean, st = stack(W, M, x, flags), stack(Wi, Mi, x, flags)
        t, y = st.inputs_t[0], st.maps_t[0]["Y"]
        torch.cuda.synchronize()
        assert int(t["n_fired"]) == T and torch.equal(y[:, rest], clean.maps_t[0]["Y"][:, rest])
        if flags:
            _same_infinities(y[:, 5], Xb[:, 7].float())
            assert torch.equal(y[:, 9], clean.maps_t[0]["Y"][:, 9])  # (a fired token does not read the image)
        else:
            _same_infinities(y[:, 5], t["R"][:, 7])
            _same_infinities(y[:, 9], t["C"][:, 3])
            assert torch.equal(gsi.gated_linear(Wi, Mi, t["C"], t["R"], t["fired_idx"], t["n_fired"]), y)
    dense, clean = gsi.dense_linear(Wi, Xb), gsi.dense_linear(W, Xb)
    _same_infinities(dense[:, 5], Xb[:, 7].float())
    assert torch.equal(dense[:, rest], clean[:, rest])
    c, clean = gsi.project(Ui, X)[0], gsi.project(U, X)[0]
    cols = [j for j in range(k) if j != 11]
    _same_infinities(c[:, 11], X[:, 17])
    assert torch.equal(c[:, cols], clean[:, cols])
