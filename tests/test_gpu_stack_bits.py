"""One token: an input's results are the same bits in a call of its own and beside any number of others."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# column blocks of a call of its own and fewer of them in a larger one: ranks that are cut evenly, raggedly (one piece more in
# the last block: 264) and not at all; slabs whose rows fill the row groups, or do not (2576: 81 rows), a last slab of few rows
# (4097); 16 inputs make whole rows, 64 KB of LDS at rank 512; widths of whole units of W r beside widths with a rest.  An
# image that is not 16-byte aligned has the projections run by themselves.
@pytest.mark.parametrize("k,dtype,widths", [
    (200, "bf16", (4096, 1024)), (256, "bf16", (4096, 16384)), (512, "bf16", (4096, 2048)), (264, "bf16", (4097, 2576)),
    (128, "bf16", (1032, 4096)), (64, "bf16", (4096, 1024)), (64, "f32", (2048, 768)), (256, "f32", (2048, 2577)), (252, "f32", (4096,)), (100, "f32", (1160,))])
@pytest.mark.parametrize("n,odd_image", [(2, False), (4, False), (6, False), (9, False), (12, False), (16, False), (6, True), (16, True)])
def test_stack_of_one_token(k, dtype, widths, n, odd_image):
    from paper_2605_03109_amd import gsi

    print(f"case stack bits k={k} {dtype} widths={widths} n={n} odd_image={odd_image}", flush=True)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator(device="cuda").manual_seed(k + n)
    inputs, maps = [], []
    for i in range(n):
        d = widths[i % len(widths)]
        U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).to(dt)
        W = (torch.randn(24, d, generator=g, device="cuda") / d**0.5).to(dt)
        flat = torch.empty(24 * k + 1, device="cuda", dtype=dt)
        M = flat[1:].view(24, k) if odd_image else flat[:-1].view(24, k)
        M.copy_(W.double() @ U.double())
        inputs.append({"U": U, "X": torch.randn(1, d, generator=g, device="cuda")})
        maps.append({"W": W, "M": M, "input_id": i})
    eps = 0.5
    st = gsi.layer_stack(inputs, maps, 1, eps)
    torch.cuda.synchronize()
    for t, mp in zip(st.inputs_t, st.maps_t):
        C, R, rn, xn = gsi.project(t["U"], t["X"])
        mask, idx, nf = gsi.gate(rn, xn, eps)
        Y = gsi.gated_linear(mp["W"], mp["M"], C, R, idx, nf)
        torch.cuda.synchronize()
        for a, b in ((C, t["C"]), (R, t["R"]), (rn, t["rnorm"]), (xn, t["xnorm"]), (mask, t["mask"]), (nf, t["n_fired"])):
            assert torch.equal(a, b)
        assert torch.equal(Y, mp["Y"])


# many tokens: whether a basis is transposed first follows from the longest input of the call; the order of the sums does not
@pytest.mark.parametrize("B,xdtype", [(900, "bf16"), (1600, "bf16"), (900, "f32")])
def test_stack_of_many_tokens(B, xdtype):
    from paper_2605_03109_amd import gsi

    print(f"case stack bits {B} tokens {xdtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(B)
    inputs, maps = [], []
    for i, (d, k) in enumerate([(1024, 256), (8256, 64), (4096, 512)]):
        U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).bfloat16()
        W = (torch.randn(136, d, generator=g, device="cuda") / d**0.5).bfloat16()
        X = torch.randn(B, d, generator=g, device="cuda").to({"bf16": torch.bfloat16, "f32": torch.float32}[xdtype])
        inputs.append({"U": U, "X": X})
        maps.append({"W": W, "M": (W.double() @ U.double()).bfloat16(), "input_id": i})
    st = gsi.layer_stack(inputs, maps, B, 0.9)
    torch.cuda.synchronize()
    for t, mp in zip(st.inputs_t, st.maps_t):
        C, R, rn, xn = gsi.project(t["U"], t["X"])
        mask, idx, nf = gsi.gate(rn, xn, 0.9)
        Y = gsi.gated_linear(mp["W"], mp["M"], C, R, idx, nf)
        torch.cuda.synchronize()
        for a, b in ((C, t["C"]), (R, t["R"]), (rn, t["rnorm"]), (xn, t["xnorm"]), (mask, t["mask"]), (Y, mp["Y"])):
            assert torch.equal(a, b)
