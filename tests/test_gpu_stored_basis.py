"""The sizes of the lines that decide whether a basis is transposed on its way or first, against the oracle's tolerances of test_gpu_image_tiles.
With the workspace that the queries name only the basis that starts 8 bytes off and fp32 tokens come to those lines, the others run on the products
that read the basis as stored; test_gpu_former_prefill brings all of them there."""
import pytest

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")

import test_gpu_image_tiles as tiles  # noqa: E402


# a work of 4096 and just above it at a rank that ends the first line, at the last rank without and the first with the second
# line; the second line's last work and just above it
@pytest.mark.parametrize("m,d,k,offset", [
    (4096, 4096, 512, 0), (4097, 4096, 512, 0), (8193, 4096, 64, 0), (8193, 4096, 192, 0), (8193, 4096, 200, 0), (16384, 4096, 200, 4),
    (16385, 4096, 200, 0),
    # 2^19 elements, whose parts are added past the caches, and just above
    (8192, 4096, 64, 0), (2048, 2048, 256, 0), (2049, 2048, 256, 0)])
def test_images(m, d, k, offset):
    tiles.test_images(m, d, k, offset)


# bf16 tokens: 1536 and one more, and 768 and one more where the input is longer than 8192
@pytest.mark.parametrize("d,k,B,xdtype", [
    (1024, 320, 1536, "bf16"), (1024, 320, 1537, "bf16"), (8192, 64, 769, "bf16"), (8256, 64, 768, "bf16"), (8256, 64, 769, "bf16"),
    (8256, 64, 1540, "f32")])
def test_coefficients(d, k, B, xdtype):
    tiles.test_coefficients(d, k, B, xdtype)
