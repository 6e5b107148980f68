"""Prefill-sized products whose operands go from memory to LDS without registers, at the edges of their tiles: the W term over the
fired rows (row tiles of up to 256 rows in steps of 16, column tiles of 256, one k-tile and odd numbers of them, parts)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# one k-tile (which takes many rows); an odd number; odd in parts; column tiles by the eight, ragged
@pytest.mark.parametrize("d,m,B", [(64, 2048, 33000), (2112, 2308, 1000), (4160, 4000, 530), (2048, 4096, 4400)])
def test_fired_rows(d, m, B):
    from paper_2605_03109_amd import gsi

    k = 64
    g = torch.Generator(device="cuda").manual_seed(d + m + B)
    R, C = torch.randn(B, d, generator=g, device="cuda"), torch.randn(B, k, generator=g, device="cuda")
    W = (torch.randn(m, d, generator=g, device="cuda") / d**0.5).to(torch.bfloat16)
    M = (torch.randn(m, k, generator=g, device="cuda") / k**0.5).to(torch.bfloat16)
    need = gsi.workspace_bytes(gsi.CALL_GATED_LINEAR, m, d, k, B)
    ws = torch.full((2 * need + (16 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    base, wr = C.double() @ M.double().T, R.to(torch.bfloat16).double() @ W.double().T
    # 32-bit sums of d exact products, and of k products of operands of 16 mantissa bits: 2^-16 of the norms that bound them
    bar = 2.0**-16 * (C.double().norm(dim=1).max() * M.double().norm(dim=1).max() + R.double().norm(dim=1).max() * W.double().norm(dim=1).max())
    for n in sorted({1, 16, 17, 128, 129, 144, 255, 256, 257, 273, 511, 513, min(B, 4353), min(B, 5000)}):
        print(f"case fired rows d={d} m={m} B={B} fired={n}", flush=True)
        fired = torch.randperm(B, generator=g, device="cuda")[:n].sort().values
        idx = torch.zeros(B, dtype=torch.int32, device="cuda")
        idx[:n] = fired.int()
        want = base.clone()
        want[fired] += wr[fired]
        count = torch.tensor([n], dtype=torch.int32, device="cuda")
        Y = torch.full((B, m), float("nan"), device="cuda")
        rc = gsi.lib.gsi_gated_linear(W.data_ptr(), M.data_ptr(), C.data_ptr(), R.data_ptr(), idx.data_ptr(), count.data_ptr(), m, d, k, B,
                                      gsi.GSI_BF16, Y.data_ptr(), gsi.GSI_F32, ws.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert rc == gsi.GSI_OK, gsi.last_error()
        assert (Y.double() - want).abs().max() <= bar
        assert bool((ws[need:] == 0x5A).all())


# one token over a row tile; column tiles that are ragged, less than one, by the eight; ranks of two k-tiles, and of six
@pytest.mark.parametrize("xdtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,k,m,B", [(64, 64, 260, 129), (320, 64, 1000, 255), (2048, 192, 2048, 256), (4160, 128, 36, 385), (1024, 256, 4100, 1030)])
def test_two_terms(d, k, m, B, xdtype):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(d + k + B)
    U = torch.linalg.qr(torch.randn(d, k, generator=g, device="cuda").double()).Q.to(torch.bfloat16).contiguous()
    X = torch.randn(B, d, generator=g, device="cuda").to(xdtype)
    W = (torch.randn(m, d, generator=g, device="cuda") / d**0.5).to(torch.bfloat16)
    M = (W.double() @ U.double()).to(torch.bfloat16)
    M[7, 0], M[8, :] = float("inf"), float("nan")  # stay in their columns of Y
    print(f"case two terms d={d} k={k} m={m} B={B} x {xdtype}", flush=True)
    st = gsi.LayerStack([{"U": U, "X": X}], [{"W": W, "M": M, "input_id": 0}], B, 2.0)  # no residual is twice its token: none fires
    st.run()
    torch.cuda.synchronize()
    t = st.inputs_t[0]
    C, x = t["C"].double(), X.double()
    # of the stored C: 16 mantissa bits of it, 32-bit sums of k products, one subtraction
    bar = lambda b: 2.0**-16 * C.norm(dim=1)[:, None] * b.double().norm(dim=1)[None, :]
    Y, rest = st.maps_t[0]["Y"], [j for j in range(m) if j not in (7, 8)]
    assert ((Y.double() - C @ M.double().T).abs() <= bar(M))[:, rest].all()
    assert not Y[:, 7].isfinite().any() and Y[:, 8].isnan().all()
    y = gsi.gated_linear(W, M, t["C"], t["R"], t["fired_idx"], t["n_fired"])
    assert torch.equal(y.view(torch.int32), Y.view(torch.int32))
    assert ((t["R"].double() - (x - C @ U.double().T)).abs() <= bar(U) + 2.0**-23 * x.abs()).all()
    # norms of the stored rows: 32-bit sums of d squares
    for got, rows in ((t["rnorm"], t["R"].double()), (t["xnorm"], x)):
        assert ((got.double() - rows.norm(dim=1)).abs() <= 2.0**-20 * rows.norm(dim=1)).all()
    assert int(t["n_fired"][0]) == 0
