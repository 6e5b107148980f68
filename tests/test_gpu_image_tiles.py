"""Images and coefficients with the basis transposed on its way to LDS, at the edges of tiles, parts and alignments."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _basis(d, k, offset, g):
    """U[d, k] in bf16 whose memory starts `offset` elements behind a 256-byte boundary."""
    flat = torch.empty(d * k + offset, device="cuda", dtype=torch.bfloat16)
    U = flat[offset:].view(d, k)
    U.copy_(torch.randn(d, k, generator=g, device="cuda") / d**0.5)
    return U


# tiles of 64 rows in many parts and in one, a row short of and past a tile; tiles of 128 and 256 rows; columns short of,
# equal to and past a tile; bases that start 8 bytes (as stored) and 2 bytes (transposed first) off
@pytest.mark.parametrize("m,d,k,offset", [
    (1, 64, 4, 0), (63, 4096, 60, 0), (65, 16384, 256, 0), (4096, 1024, 260, 4), (300, 10240, 512, 0), (16384, 512, 256, 0),
    (16321, 320, 64, 4), (1024, 5120, 256, 0), (1025, 5120, 256, 4), (300, 13632, 300, 0), (16384, 4096, 256, 0), (16385, 4096, 256, 0), (33000, 192, 128, 0), (70000, 256, 256, 0), (65, 1024, 68, 1), (33000, 128, 64, 1)])
def test_images(m, d, k, offset):
    from paper_2605_03109_amd import gsi

    print(f"case image m={m} d={d} k={k} offset={offset}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + d + k)
    W = torch.randn(m, d, generator=g, device="cuda").bfloat16()
    U = _basis(d, k, offset, g)
    need = gsi.workspace_bytes(gsi.CALL_BUILD_IMAGE, m, d, k, 0)
    ws = torch.empty(need + 4096, device="cuda", dtype=torch.uint8).fill_(255)
    M = gsi.build_image(W, U, ws=ws[:need])
    torch.cuda.synchronize()
    assert (ws[need:] == 255).all()  # nothing behind the workspace that the query names
    ref = torch.cat([W[i:i + 4096].double() @ U.double() for i in range(0, m, 4096)])
    mag = torch.cat([W[i:i + 4096].double().abs() @ U.double().abs() for i in range(0, m, 4096)])
    # half a unit in the last place of bf16, and fp32 sums of d terms
    bound = ref.abs() * 2**-8 + mag * (8 + d**0.5) * 2**-24
    assert ((M.double() - ref).abs() <= bound).all()


# the last and the first side of the rule, both activation types, one and two column tiles, a ragged last row tile
@pytest.mark.parametrize("d,k,B,xdtype", [
    (1024, 64, 129, "bf16"), (1024, 320, 1000, "f32"), (1024, 320, 1024, "bf16"), (1024, 320, 1025, "bf16"), (1088, 192, 1100, "f32"),
    (16384, 512, 200, "bf16"), (4096, 128, 300, "f32")])
def test_coefficients(d, k, B, xdtype):
    from paper_2605_03109_amd import gsi

    print(f"case coefficients d={d} k={k} B={B} {xdtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(d + k + B)
    U = _basis(d, k, 0, g)
    X = torch.randn(B, d, generator=g, device="cuda").to({"f32": torch.float32, "bf16": torch.bfloat16}[xdtype])
    C, R, rn, xn = gsi.project(U, X)
    torch.cuda.synchronize()
    ref = X.double() @ U.double()
    mag = X.double().abs() @ U.double().abs()
    # fp32 sums of d terms, a head and a tail of 2^-17
    assert ((C.double() - ref).abs() <= mag * ((8 + d**0.5) * 2**-24 + (2**-17 if xdtype == "f32" else 0))).all()
    assert torch.linalg.norm(R.double() - (X.double() - ref @ U.double().T)) <= 2e-5 * torch.linalg.norm(X.double())
