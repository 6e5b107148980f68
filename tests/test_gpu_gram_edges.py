"""E = U^T U - I at the edges of its tiles and chunks: column tails, row tails, bases without 16-byte alignment."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,k,dt,shift", [(1003, 24, "bf16", 0), (31, 8, "bf16", 0), (530, 72, "bf16", 0), (530, 72, "bf16", 1),
                                          (17, 4, "f32", 0), (515, 20, "f32", 0), (515, 20, "f32", 1), (3, 1, "f32", 0)])
def test_gram_tiles(d, k, dt, shift):
    from paper_2605_03109_amd import gsi

    gen = torch.Generator().manual_seed(7 * d + k)
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    flat = torch.zeros(d * k + 8, dtype=dtype, device="cuda")
    U = flat[shift:shift + d * k].view(d, k)  # shift 1: two or four bytes past a 16-byte boundary
    U.copy_((torch.randn((d, k), generator=gen) / d**0.5).to(dtype))
    print(f"case gram d={d} k={k} {dt} shift={shift}", flush=True)
    E = gsi.build_gram(U).cpu().double().numpy()
    u = U.cpu().double().numpy()
    ref = u.T @ u - np.eye(k)
    # fp64 sums, one rounding to fp32
    assert np.all(np.abs(E - ref) <= 2.0**-24 * np.abs(ref) + 1e-13)
    assert np.array_equal(E, E.T)
