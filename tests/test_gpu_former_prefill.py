"""Prefill-sized calls that bring exactly the workspace that the queries named before operands were laid out as bf16 in it, and images whose basis
is aligned to 8 bytes only: served by the kernels that read c, r and the basis as they are, on both sides of the lines between these."""
import pytest
import torch

import test_gpu_image_tiles as tiles

pytestmark = pytest.mark.gpu


def _rows(g, *s):
    return torch.randn(*s, generator=g, device="cuda")


# bf16 tokens: the basis as stored up to 1536, or 768 where the input is longer than 8192, transposed first beyond; fp32 tokens
@pytest.mark.parametrize("d,k,B,former,xdtype", [
    (1024, 320, 1536, 4784128, torch.bfloat16), (1024, 320, 1537, 4786944, torch.bfloat16), (8192, 256, 769, 17581056, torch.bfloat16),
    (8256, 192, 768, 11040768, torch.bfloat16), (8256, 192, 769, 11051264, torch.bfloat16), (1024, 320, 2000, 6031360, torch.float32),
    (4160, 512, 400, 11021568, torch.float32), (1088, 192, 257, 847616, torch.bfloat16)])
def test_projection(d, k, B, former, xdtype):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(d + k + B)
    U = torch.linalg.qr(_rows(g, d, k).double()).Q.to(torch.bfloat16).contiguous()
    X = _rows(g, B, d).to(xdtype)
    print(f"case former projection d={d} k={k} B={B} x {xdtype}", flush=True)
    assert former < gsi.workspace_bytes(gsi.CALL_PROJECT, 0, d, k, B)
    ws = torch.full((former + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    C, R = torch.empty(B, k, device="cuda"), torch.empty(B, d, device="cuda")
    rn, xn = torch.empty(B, device="cuda"), torch.empty(B, device="cuda")
    rc = gsi.lib.gsi_project(U.data_ptr(), X.data_ptr(), d, k, B, gsi.GSI_BF16, gsi.dtype_code(X), C.data_ptr(), R.data_ptr(), rn.data_ptr(), xn.data_ptr(),
                             ws.data_ptr(), former, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == gsi.GSI_OK, gsi.last_error()
    x, u, c = X.double(), U.double(), C.double()
    # head and tail of fp32 tokens leave 2^-18 of them (half a unit of bf16, twice); 32-bit sums of d products, or 2 d
    rel = (8 + d**0.5) * 2.0**-24 if xdtype == torch.bfloat16 else 2.0**-17 + (8 + (2 * d) ** 0.5) * 2.0**-24
    assert ((c - x @ u).abs() <= rel * (x.abs() @ u.abs())).all()
    # of the stored C: 16 mantissa bits of it, 32-bit sums of k products, one subtraction; norms of the stored rows, 32-bit sums of d squares
    assert ((R.double() - (x - c @ u.T)).abs() <= 2.0**-16 * c.norm(dim=1)[:, None] * u.norm(dim=1)[None, :] + 2.0**-23 * x.abs()).all()
    for got, rows in ((rn, R.double()), (xn, x)):
        assert ((got.double() - rows.norm(dim=1)).abs() <= 2.0**-20 * rows.norm(dim=1)).all()
    assert bool((ws[former:] == 0x5A).all())


# the basis transposed on its way to LDS, or first: a work of 4096 and just above it, at a rank that ends the first line, at the last rank without and
# the first with the second line; the second line's last work and just above it; parts added past the caches and not
@pytest.mark.parametrize("m,d,k", [(4096, 4096, 512), (4097, 4096, 512), (8193, 4096, 64), (8193, 4096, 192), (8193, 4096, 200), (16384, 4096, 200), (16385, 4096, 200),
                                   (8192, 4096, 64), (2048, 2048, 256), (2049, 2048, 256)])
def test_images(m, d, k):
    tiles.test_images(m, d, k, 4)


# W r of r as it is, and the image term of c as it is: one tile of fired rows and several, parts, column tiles with remainders
@pytest.mark.parametrize("m,d,k,B,former", [(2308, 2112, 64, 1000, 36928000), (4096, 4096, 64, 600, 39321600), (4100, 1024, 128, 700, 4198400),
                                            (1000, 16384, 256, 2048, 65536000)])
def test_gated_map(m, d, k, B, former):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(m + d + k + B)
    R, C = _rows(g, B, d), _rows(g, B, k)
    W, M = (_rows(g, m, d) / d**0.5).to(torch.bfloat16), (_rows(g, m, k) / k**0.5).to(torch.bfloat16)
    assert former < gsi.workspace_bytes(gsi.CALL_GATED_LINEAR, m, d, k, B)
    ws = torch.full((former + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    base, wr = C.double() @ M.double().T, R.to(torch.bfloat16).double() @ W.double().T
    # 32-bit sums of d exact products, and of k products of operands of 16 mantissa bits: 2^-16 of the norms that bound them
    bar = 2.0**-16 * (C.double().norm(dim=1).max() * M.double().norm(dim=1).max() + R.double().norm(dim=1).max() * W.double().norm(dim=1).max())
    for n in (0, 1, 17, 129, 300, B):
        print(f"case former map m={m} d={d} k={k} B={B} fired={n}", flush=True)
        idx = torch.zeros(B, dtype=torch.int32, device="cuda")
        fired = torch.randperm(B, generator=g, device="cuda")[:n].sort().values
        idx[:n] = fired.int()
        want = base.clone()
        want[fired] += wr[fired]
        count = torch.tensor([n], dtype=torch.int32, device="cuda")
        Y = torch.full((B, m), float("nan"), device="cuda")
        rc = gsi.lib.gsi_gated_linear(W.data_ptr(), M.data_ptr(), C.data_ptr(), R.data_ptr(), idx.data_ptr(), count.data_ptr(), m, d, k, B, gsi.GSI_BF16, Y.data_ptr(),
                                      gsi.GSI_F32, ws.data_ptr(), former, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert rc == gsi.GSI_OK, gsi.last_error()
        assert (Y.double() - want).abs().max() <= bar
        assert bool((ws[former:] == 0x5A).all())


# residual rows and image terms of c as it is in one launch, and the W terms behind them
@pytest.mark.parametrize("shape,maps,B,former,xdtype", [
    ([(1024, 256), (2048, 256)], [(1024, 0), (2048, 0), (1024, 1)], 1601, 77601280, torch.bfloat16),
    ([(1024, 256), (4096, 256)], [(1024, 0), (4096, 0), (1024, 1)], 700, 61847040, torch.float32)])
def test_block(shape, maps, B, former, xdtype):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(B)
    inputs, mp, fired = [], [], B // 5
    for d, k in shape:
        U = torch.linalg.qr(_rows(g, d, k)).Q.to(torch.bfloat16).contiguous()
        X = _rows(g, B, k) @ U.float().T
        X[torch.randperm(B, generator=g, device="cuda")[:fired]] += 0.5 * _rows(g, fired, d)
        inputs.append({"U": U, "X": X.to(xdtype).contiguous()})
    for m, i in maps:
        W = (_rows(g, m, shape[i][0]) / shape[i][0]**0.5).to(torch.bfloat16)
        mp.append({"W": W, "M": (W.float() @ inputs[i]["U"].float()).to(torch.bfloat16), "input_id": i})
    print(f"case former block {shape} B={B} x {xdtype}", flush=True)
    st = gsi.LayerStack(inputs, mp, B, 0.1)
    ws = torch.full((former + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    assert former < st.ws.numel()
    st.ws = ws[:former]
    st.run()
    torch.cuda.synchronize()
    assert bool((ws[former:] == 0x5A).all())
    for t, mt in ((st.inputs_t[q["input_id"]], q) for q in st.maps_t):
        C, R, U, x = t["C"].double(), t["R"].double(), t["U"].double(), t["X"].double()
        assert int(t["n_fired"][0]) == fired
        assert ((R - (x - C @ U.T)).abs() <= 2.0**-16 * C.norm(dim=1)[:, None] * U.norm(dim=1)[None, :] + 2.0**-23 * x.abs()).all()
        want = C @ mt["M"].double().T
        rows = t["fired_idx"][:fired].long()
        want[rows] += t["R"][rows].to(torch.bfloat16).double() @ mt["W"].double().T
        bar = 2.0**-16 * (C.norm(dim=1).max() * mt["M"].double().norm(dim=1).max() + R.norm(dim=1).max() * mt["W"].double().norm(dim=1).max())
        assert (mt["Y"].double() - want).abs().max() <= bar
