"""Prefill calls of more bytes than the memory-side cache holds: rows past the caches hold what rows through them hold."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# both forms of a fired token's product, both types of x (three operand forms); a last tile of two rows; all tokens fire, some
# parts of a product then have no rows to add, or none does
@pytest.mark.parametrize("xdtype", ["bf16", "f32"])
@pytest.mark.parametrize("wx", [False, True])
@pytest.mark.parametrize("eps", [1e-3, 0.9922, 10.0])
def test_large_calls(xdtype, wx, eps):
    from paper_2605_03109_amd import gsi

    print(f"case past caches x={xdtype} wx={wx} eps={eps}", flush=True)
    B, k = 130, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    inputs, maps = [], []
    for i, (d, m) in enumerate([(4096, 16384), (16384, 4096)]):  # weights of 268 MB together, 134 MB each
        U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).bfloat16()
        W = (torch.randn(m, d, generator=g, device="cuda") / d**0.5).bfloat16()
        X = torch.randn(B, d, generator=g, device="cuda").to({"f32": torch.float32, "bf16": torch.bfloat16}[xdtype])
        inputs.append({"U": U, "X": X, "flags": gsi.INPUT_SLOW_PATH_WX if wx else 0})
        maps.append({"W": W, "M": (W.float() @ U.float()).bfloat16(), "input_id": i})
    both = gsi.layer_stack(inputs, maps, B, eps)
    torch.cuda.synchronize()
    if eps == 0.9922:  # (|r| / |x| of tokens of 4096 is about (1 - 64 / 4096)^0.5, on both sides of it)
        assert any(0 < int(t["n_fired"]) < B for t in both.inputs_t)
    for i in range(2):
        one = gsi.layer_stack([inputs[i]], [{**maps[i], "input_id": 0}], B, eps)
        torch.cuda.synchronize()
        for name in ("C", "R", "rnorm", "xnorm", "mask", "n_fired"):
            assert torch.equal(one.inputs_t[0][name], both.inputs_t[i][name]), name
        assert torch.equal(one.maps_t[0]["Y"], both.maps_t[i]["Y"])


def test_large_projection():
    from paper_2605_03109_amd import gsi

    d, k, B = 16384, 64, 4097  # R and x: 403 MB
    print(f"case past caches projection d={d} k={k} B={B}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(4)
    U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).bfloat16()
    X = torch.randn(B, d, generator=g, device="cuda").bfloat16()
    C, R, rn, xn = gsi.project(U, X)
    torch.cuda.synchronize()
    for rows in (slice(0, 256), slice(B - 130, B)):
        x = X[rows].double()
        r = x - (x @ U.double()) @ U.double().T
        # fp32 sums of d terms (c, head and tail of which enter the second product with 2^-17) and of k terms
        assert torch.linalg.norm(R[rows].double() - r) <= 2e-5 * torch.linalg.norm(x)
        assert torch.allclose(rn[rows].double(), torch.linalg.norm(r, dim=1), rtol=1e-5)
        assert torch.allclose(xn[rows].double(), torch.linalg.norm(x, dim=1), rtol=1e-5)
