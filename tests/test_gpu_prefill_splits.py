"""Split contractions of prefill-sized products: every number of parts that the rule gives, one row tile and several, with the
workspace that the query names and with the sizes that it named before; a dense stack equals its separate products."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _operands(d, m, B, xdtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return r(B, d).to(xdtype), (r(m, d) / d**0.5).to(torch.bfloat16)


def _dense(gsi, W, X, nbytes):
    m, d = W.shape
    Y = torch.full((X.shape[0], m), float("nan"), device="cuda")
    ws = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    rc = gsi.lib.gsi_dense_linear(W.data_ptr(), X.data_ptr(), m, d, X.shape[0], gsi.GSI_BF16, gsi.dtype_code(X), Y.data_ptr(),
                                  ws.data_ptr() if nbytes else None, nbytes, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return rc, Y


# 32 tiles in 4 parts, in 2; 40 in 2; 64 in 4; 128 in 2; a long contraction in 16; a ragged last tile
@pytest.mark.parametrize("xdtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,m,B", [(4096, 4096, 129), (1024, 4096, 200), (2560, 5000, 140), (4096, 4096, 400), (2048, 8192, 500),
                                   (8192, 260, 300), (4096, 3000, 333)])
def test_dense_products(d, m, B, xdtype):
    from paper_2605_03109_amd import gsi

    X, W = _operands(d, m, B, xdtype, d + m + B)
    print(f"case split dense d={d} m={m} B={B} {xdtype}", flush=True)
    want = X.double() @ W.double().T
    # operands of 16 mantissa bits (two bf16 terms), 32-bit sums of d products: 2^-16 of the norms that bound the sum
    bar = 2.0**-16 * X.double().norm(dim=1).max() * W.double().norm(dim=1).max()
    full = gsi.workspace_bytes(gsi.CALL_DENSE_LINEAR, m, d, 0, B)
    rc, Y = _dense(gsi, W, X, full)
    assert rc == gsi.GSI_OK and (Y.double() - want).abs().max() <= bar
    st = gsi.LayerStack([{"U": torch.zeros(d, 64, dtype=torch.bfloat16, device="cuda"), "X": X}],
                        [{"W": W, "M": torch.zeros(m, 64, dtype=torch.bfloat16, device="cuda"), "input_id": 0}] * 2, B, 0.1)
    st.run_dense()
    torch.cuda.synchronize()
    assert torch.equal(st.maps_t[0]["Y"], Y) and torch.equal(st.maps_t[1]["Y"], Y)


# (d, m, B): sizes that the query named before; a call that brings less than it names now is split less
@pytest.mark.parametrize("d,m,B,sizes", [(4096, 4096, 129, (16908288, 0)), (4096, 4096, 400, (52428800, 0)),
                                         (8192, 260, 300, (4992000, 2496000))])
def test_former_workspaces(d, m, B, sizes):
    from paper_2605_03109_amd import gsi

    X, W = _operands(d, m, B, torch.bfloat16, d + m + B)
    want = X.double() @ W.double().T
    bar = 2.0**-16 * X.double().norm(dim=1).max() * W.double().norm(dim=1).max()
    for nbytes in sizes:
        print(f"case former workspace d={d} m={m} B={B} bytes={nbytes}", flush=True)
        rc, Y = _dense(gsi, W, X, nbytes)
        assert rc == gsi.GSI_OK, (nbytes, gsi.last_error())
        assert (Y.double() - want).abs().max() <= bar


# counts below, at and above the rows that a product is sized for, one row tile and several: the parts of the contraction
# follow the count, and their sums stay inside the workspace that the query names (33 to 512 rows are sized as one tile of
# 128, 2048 as four; 640 as two)
@pytest.mark.parametrize("d,k,m,B", [(1024, 64, 260, 129), (4096, 64, 1000, 257), (2560, 128, 5000, 300), (4096, 64, 8192, 640),
                                     (4096, 64, 10240, 2048), (8192, 64, 260, 1000)])
def test_fired_counts(d, k, m, B):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(d + m + B)
    R, C = torch.randn(B, d, generator=g, device="cuda"), torch.randn(B, k, generator=g, device="cuda")
    W = (torch.randn(m, d, generator=g, device="cuda") / d**0.5).to(torch.bfloat16)
    M = (torch.randn(m, k, generator=g, device="cuda") / k**0.5).to(torch.bfloat16)
    need = gsi.workspace_bytes(gsi.CALL_GATED_LINEAR, m, d, k, B)
    guard = 4 * need + (64 << 20)  # what parts of a row tile more than there is would reach
    ws = torch.full((need + guard,), 0x5A, dtype=torch.uint8, device="cuda")
    base, wr = C.double() @ M.double().T, R.to(torch.bfloat16).double() @ W.double().T
    # 32-bit sums of d exact products, and of k products of operands of 16 mantissa bits: 2^-16 of the norms that bound them
    bar = 2.0**-16 * (C.double().norm(dim=1).max() * M.double().norm(dim=1).max() + R.double().norm(dim=1).max() * W.double().norm(dim=1).max())
    for n in sorted({0, 1, 127, 128, 129, B // 4, B // 2, B - 1, B}):
        print(f"case fired count d={d} m={m} B={B} fired={n}", flush=True)
        fired = torch.randperm(B, generator=g, device="cuda")[:n].sort().values
        idx = torch.zeros(B, dtype=torch.int32, device="cuda")
        idx[:n] = fired.int()
        want = base.clone()
        want[fired] += wr[fired]
        count = torch.tensor([n], dtype=torch.int32, device="cuda")
        ys = []
        for _ in range(2):
            Y = torch.full((B, m), float("nan"), device="cuda")
            rc = gsi.lib.gsi_gated_linear(W.data_ptr(), M.data_ptr(), C.data_ptr(), R.data_ptr(), idx.data_ptr(), count.data_ptr(),
                                          m, d, k, B, gsi.GSI_BF16, Y.data_ptr(), gsi.GSI_F32, ws.data_ptr(), need,
                                          torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert rc == gsi.GSI_OK, gsi.last_error()
            ys.append(Y)
        assert torch.equal(ys[0], ys[1]) and (ys[0].double() - want).abs().max() <= bar
        assert bool((ws[need:] == 0x5A).all())
