"""Images and coefficients of prefill-sized calls on the products that read the basis as stored: ranks that are no multiple of the column
tile or of a fragment, row tiles and column tiles with remainders, contractions of one k-tile, of an odd number, in parts, and shorter
than the tiles on their way."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,k", [(64, 192, 136), (63, 256, 192), (130, 320, 256), (1000, 1088, 200), (68, 1024, 264), (4096, 4096, 256),
                                   (257, 2048, 512), (1028, 8256, 144), (16384, 1024, 256),
                                   # one fragment of columns and less; tiles of 128 rows in parts, unsplit, the last before two rounds of them
                                   (64, 64, 8), (200, 320, 24), (2600, 8192, 520), (16500, 192, 64), (65400, 256, 16), (12400, 4160, 136)])
def test_image(m, d, k):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(m + d + k)
    W = torch.randn(m, d, generator=g, device="cuda").to(torch.bfloat16)
    U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).to(torch.bfloat16)
    U[3, 5], U[d - 1, k - 1] = float("inf"), float("nan")   # stay in their columns
    print(f"case image m={m} d={d} k={k}", flush=True)
    need = gsi.workspace_bytes(gsi.CALL_BUILD_IMAGE, m, d, k, 0)
    ws = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    M = torch.full((m + 1, k), 7.0, dtype=torch.bfloat16, device="cuda")
    rc = gsi.lib.gsi_build_image(W.data_ptr(), U.data_ptr(), M.data_ptr(), m, d, k, gsi.GSI_BF16, ws.data_ptr(), need,
                                 torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == gsi.GSI_OK, gsi.last_error()
    rest = [j for j in range(k) if j not in (5, k - 1)]
    w, u = W.double(), U.double()[:, rest]
    want, got = w @ u, M[:m, rest].double()
    # one rounding to bf16, 32-bit sums of d exact products
    bar = 2.0**-8 * want.abs() + (8 + d**0.5) * 2.0**-24 * (w.abs() @ u.abs())
    assert ((got - want).abs() <= bar).all()
    assert not M[:m, 5].isfinite().any() and M[:m, k - 1].isnan().all()
    assert bool((M[m] == 7.0).all()) and bool((ws[need:] == 0x5A).all())


# a workspace of the size that the query named before is served as it was, and gives the same to rounding
@pytest.mark.parametrize("m,d,k,former", [(64, 2560, 16, 98304), (64, 6144, 512, 7340032)])
def test_image_in_a_former_workspace(m, d, k, former):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(m + d + k)
    W = torch.randn(m, d, generator=g, device="cuda").to(torch.bfloat16)
    U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).to(torch.bfloat16)
    print(f"case image in a former workspace m={m} d={d} k={k}", flush=True)
    ws = torch.full((former + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    M = torch.empty(m, k, dtype=torch.bfloat16, device="cuda")
    rc = gsi.lib.gsi_build_image(W.data_ptr(), U.data_ptr(), M.data_ptr(), m, d, k, gsi.GSI_BF16, ws.data_ptr(), former,
                                 torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == gsi.GSI_OK, gsi.last_error()
    w, u = W.double(), U.double()
    want = w @ u
    assert ((M.double() - want).abs() <= 2.0**-8 * want.abs() + (8 + d**0.5) * 2.0**-24 * (w.abs() @ u.abs())).all()
    assert bool((ws[former:] == 0x5A).all())


# one row over a tile of 128; one k-tile, an odd number; many parts of four k-tiles, of eight, of unequal length; column tiles with remainders
@pytest.mark.parametrize("d,k,B", [(64, 64, 129), (192, 128, 300), (1088, 192, 257), (4096, 64, 140), (2048, 320, 640), (16384, 256, 385),
                                   (10240, 64, 640), (4160, 512, 400), (16384, 512, 700)])
def test_coefficients(d, k, B):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(d + k + B)
    X = torch.randn(B, d, generator=g, device="cuda").to(torch.bfloat16)
    U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).to(torch.bfloat16)
    print(f"case coefficients d={d} k={k} B={B}", flush=True)
    C, R, rn, xn = gsi.project(U, X)
    torch.cuda.synchronize()
    x, u = X.double(), U.double()
    # 32-bit sums of d exact products
    assert ((C.double() - x @ u).abs() <= (8 + d**0.5) * 2.0**-24 * (x.abs() @ u.abs())).all()


# fp32 activations: contractions too short to cut, at the four tiles that are cut to four k-tiles and one more, an odd number of k-tiles on
# eight and nine tiles, the most parts
@pytest.mark.parametrize("d,k,B", [(256, 64, 512), (512, 64, 129), (1024, 64, 512), (1024, 64, 513), (4160, 512, 400), (4160, 192, 1025), (16384, 64, 130),
                                   (16384, 512, 400), (10240, 64, 640), (4160, 512, 700)])
def test_coefficients_of_fp32_rows(d, k, B):
    from paper_2605_03109_amd import gsi

    g = torch.Generator(device="cuda").manual_seed(d + k + B)
    X = torch.randn(B, d, generator=g, device="cuda")
    U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).to(torch.bfloat16)
    print(f"case fp32 coefficients d={d} k={k} B={B}", flush=True)
    need = gsi.workspace_bytes(gsi.CALL_PROJECT, 0, d, k, B)
    ws = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    C, R = torch.empty(B, k, device="cuda"), torch.empty(B, d, device="cuda")
    rn, xn = torch.empty(B, device="cuda"), torch.empty(B, device="cuda")
    rc = gsi.lib.gsi_project(U.data_ptr(), X.data_ptr(), d, k, B, gsi.GSI_BF16, gsi.GSI_F32, C.data_ptr(), R.data_ptr(), rn.data_ptr(), xn.data_ptr(),
                             ws.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == gsi.GSI_OK, gsi.last_error()
    x, u = X.double(), U.double()
    # head and tail of x leave 2^-18 of it (half a unit of bf16, twice); 32-bit sums of 2 d exact products
    assert ((C.double() - x @ u).abs() <= (2.0**-17 + (8 + (2 * d) ** 0.5) * 2.0**-24) * (x.abs() @ u.abs())).all()
    assert bool((ws[need:] == 0x5A).all())
