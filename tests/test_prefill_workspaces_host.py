"""Prefill-sized calls with a workspace of the sizes that the queries named before operands were laid out as bf16 in it: served
as they were.  Decided on the host."""
import pytest

torch = pytest.importorskip("torch")

# (made-up addresses: a call that passes validation fails for want of a device, never where there is one)
pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="made-up addresses: only where nothing can be launched")

ADDR = 1 << 20


@pytest.mark.parametrize("d,k,B,former", [(4096, 64, 300, 1292288), (1024, 256, 2048, 4980736)])
def test_projection(d, k, B, former):
    from paper_2605_03109_amd import gsi

    call = lambda n: gsi.lib.gsi_project(ADDR, ADDR, d, k, B, gsi.GSI_BF16, gsi.GSI_BF16, ADDR, ADDR, ADDR, ADDR, ADDR, n, None)
    assert call(former) == gsi.GSI_ERR_HIP, gsi.last_error()
    assert call(gsi.workspace_bytes(gsi.CALL_PROJECT, 0, d, k, B)) == gsi.GSI_ERR_HIP
    assert call(256) == gsi.GSI_ERR_WORKSPACE


@pytest.mark.parametrize("m,d,k,B,former", [(4096, 4096, 64, 600, 39321600), (1000, 16384, 256, 2048, 65536000), (2048, 256, 64, 129, 0)])
def test_gated_map(m, d, k, B, former):
    from paper_2605_03109_amd import gsi

    call = lambda ws, n: gsi.lib.gsi_gated_linear(ADDR, ADDR, ADDR, ADDR, ADDR, ADDR, m, d, k, B, gsi.GSI_BF16, ADDR, gsi.GSI_F32, ws, n, None)
    assert call(ADDR if former else None, former) == gsi.GSI_ERR_HIP, gsi.last_error()
    full = gsi.workspace_bytes(gsi.CALL_GATED_LINEAR, m, d, k, B)
    assert full > former and call(ADDR, full) == gsi.GSI_ERR_HIP


@pytest.mark.parametrize("m,d,k,former", [(64, 2560, 16, 98304), (64, 10240, 16, 376832), (64, 6144, 512, 7340032)])
def test_image(m, d, k, former):
    from paper_2605_03109_amd import gsi

    call = lambda n: gsi.lib.gsi_build_image(ADDR, ADDR, ADDR, m, d, k, gsi.GSI_BF16, ADDR, n, None)
    assert call(former) == gsi.GSI_ERR_HIP, gsi.last_error()
    full = gsi.workspace_bytes(gsi.CALL_BUILD_IMAGE, m, d, k, 0)
    assert full > former and call(full) == gsi.GSI_ERR_HIP
