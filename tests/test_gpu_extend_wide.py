"""Basis extension at the edges of the residual's sums and of the image rows: ranks beyond what a workgroup adds up in LDS,
row tails, storage without 16-byte rows."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,K,k0,ms,dt", [(2304, 2080, 5, (17,), "bf16"), (2056, 2048, 2047, (16, 1), "bf16"), (517, 64, 3, (33,), "f32"),
                                          (520, 61, 60, (5, 64), "bf16"), (4100, 128, 0, (130,), "f32")])
def test_one_column(d, K, k0, ms, dt):
    from paper_2605_03109_amd import gsi

    gen = torch.Generator().manual_seed(d + K)
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    U = torch.zeros((d, K), dtype=dtype)
    U[:, :k0] = (torch.randn((d, k0), generator=gen) / d**0.5).to(dtype)
    x = torch.randn((1, d), generator=gen, dtype=torch.float64)
    u = U.double()
    r = (x - (x @ u) @ u.T)[0].float()
    W = [(torch.randn((m, d), generator=gen) / d**0.5).to(dtype) for m in ms]
    print(f"case extend d={d} K={K} k={k0} maps={ms} {dt}", flush=True)
    dev = lambda t: t.cuda().contiguous()
    Ud, Md = dev(U), [torch.zeros((m, K), dtype=dtype, device="cuda") for m in ms]
    Wd, E = [dev(w) for w in W], torch.zeros((K, K), device="cuda")
    kc = torch.tensor([k0], dtype=torch.int32, device="cuda")
    norm = lambda v: v.norm().float().reshape(1).cuda()
    grown = gsi.extend_basis(Ud, kc, dev(r), norm(r), norm(x), 0.05, list(zip(Wd, Md)), E)
    torch.cuda.synchronize()
    assert int(grown) == 1 and int(kc) == k0 + 1
    got = Ud.cpu()
    assert torch.equal(got[:, :k0], U[:, :k0]) and not got[:, k0 + 1:].any()
    r64 = r.double()
    r2 = r64 - u @ (u.T @ r64)
    want = r2 / r2.norm()
    # one rounding to storage (2^-8 / 2^-24 relative) of a vector known to a few 1e-6 of its length
    half_ulp = 2.0**-8 if dt == "bf16" else 2.0**-24
    col = got[:, k0].double()
    assert ((col - want).abs() <= half_ulp * want.abs() + 2e-6 * want.abs().max()).all()
    full = got.double()
    for w, M in zip(W, Md):
        m = w.double() @ col
        bound = half_ulp * m.abs() + (8 + d**0.5) * 2.0**-24 * (w.double().abs() @ col.abs())
        assert ((M.cpu()[:, k0].double() - m).abs() <= bound).all()
        assert not M.cpu()[:, :k0].any() and not M.cpu()[:, k0 + 1:].any()
    e = full.T @ col
    e[k0] -= 1.0
    assert (E.cpu()[:, k0].double() - e).abs().max() <= 2e-6 and torch.equal(E.cpu()[:, k0], E.cpu()[k0])
