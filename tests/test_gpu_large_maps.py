"""One map of at least half a gigabyte and one token: its weights stream past the caches (non-temporal loads)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# whole units of a row and a rest, a vector that the LDS holds and one that goes through it in blocks, both types; the last
# shape of each type is the same just below the limit
@pytest.mark.parametrize("m,d,k,dtype", [
    (32768, 8192, 64, "bf16"), (65544, 4104, 24, "bf16"), (8192, 32768, 64, "bf16"), (16001, 16784, 40, "bf16"), (32767, 8192, 64, "bf16"),
    (32768, 4096, 64, "f32"), (65544, 2052, 20, "f32"), (4096, 32768, 64, "f32"), (8001, 16780, 36, "f32"), (32767, 4096, 64, "f32")])
@pytest.mark.parametrize("fires", [True, False])
def test_map_past_the_caches(m, d, k, dtype, fires):
    from paper_2605_03109_amd import gsi

    print(f"case large map {m}x{d} rank {k} {dtype} fires={fires}", flush=True)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator(device="cuda").manual_seed(m + d)
    W = torch.empty(m, d, device="cuda", dtype=dt).normal_(generator=g)
    M = torch.empty(m, k, device="cuda", dtype=dt).normal_(generator=g)
    C = torch.randn(1, k, generator=g, device="cuda")
    R = torch.randn(1, d, generator=g, device="cuda")
    idx = torch.zeros(1, dtype=torch.int32, device="cuda")
    nf = torch.full((1,), int(fires), dtype=torch.int32, device="cuda")
    Y = torch.full((1, m), 7.25, device="cuda")
    got = gsi.gated_linear(W, M, C, R, idx, nf, Y=Y)
    torch.cuda.synchronize()
    y = (C.double() @ M.double().T)[0]
    scale = (C.double().square() @ M.double().square().T)[0]
    if fires:
        for r0 in range(0, m, 4096):  # (a part of W in 64 bits at a time)
            w = W[r0:r0 + 4096].double()
            y[r0:r0 + 4096] += (w @ R.double().T)[:, 0]
            scale[r0:r0 + 4096] += (w.square() @ R.double().square().T)[:, 0]
    # fp32 sums of at most k + d terms: per row, 2^-24 times the square root of their number, of the root of the terms' squares
    # (the sums on the way are no longer than that but for a factor), six of those deviations
    bound = 6 * 2**-24 * (d + k)**0.5 * scale.sqrt()
    assert got.data_ptr() == Y.data_ptr()
    assert bool(((got[0].double() - y).abs() <= bound).all())
