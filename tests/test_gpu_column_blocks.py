"""One token: the columns of a basis cut into blocks of unlike widths, against the same sums in 64 bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# four blocks of 6 and 7 pieces; two of 6 and 7; one; blocks of 6 pieces; fp32 pieces; many inputs, so that nothing is cut
@pytest.mark.parametrize("d,k,dtype,n", [
    (4096, 200, "bf16", 1), (1024, 104, "bf16", 2), (1024, 88, "bf16", 1), (2048, 192, "bf16", 4), (4096, 504, "bf16", 3),
    (1160, 100, "f32", 1), (768, 252, "f32", 2), (4096, 200, "bf16", 13)])
def test_column_blocks(d, k, dtype, n):
    from paper_2605_03109_amd import gsi

    print(f"case column blocks d={d} k={k} {dtype} inputs={n}", flush=True)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator(device="cuda").manual_seed(d + k)
    inputs, maps = [], []
    for i in range(n):
        U = torch.linalg.qr(torch.randn(d, k, generator=g, device="cuda", dtype=torch.float64))[0].to(dt).contiguous()
        W = (torch.randn(264, d, generator=g, device="cuda") / d**0.5).to(dt)
        M = (W.double() @ U.double()).to(dt)
        inputs.append({"U": U, "X": torch.randn(1, d, generator=g, device="cuda")})
        maps.append({"W": W, "M": M, "input_id": i})
    st = gsi.layer_stack(inputs, maps, 1, 0.05)
    torch.cuda.synchronize()
    rel = lambda a, b: float(torch.linalg.norm(a.double() - b) / torch.linalg.norm(b))
    for t, m in zip(st.inputs_t, st.maps_t):
        x, U = t["X"].double(), t["U"].double()
        c = x @ U
        r = x - c @ U.T
        # fp32 sums of d (c) and k (r) terms: random-walk growth of roundings of 2^-24, four times that
        assert rel(t["C"], c) <= 4 * 2**-24 * d**0.5
        assert rel(t["R"], r) <= 4 * 2**-24 * (d**0.5 + k**0.5)
        y = c @ m["M"].double().T + r @ m["W"].double().T  # (every token fires)
        assert int(t["n_fired"]) == 1 and rel(m["Y"], y) <= 4 * 2**-24 * (d**0.5 + k**0.5)
