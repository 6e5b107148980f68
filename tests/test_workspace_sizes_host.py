"""Workspaces that calls used to be served with: none at all, unusable memory where none was needed, and the smaller sizes
that the queries named before further shapes had vector kernels.  Everything here is decided on the host."""
import pytest

torch = pytest.importorskip("torch")

# A call that passes validation goes on to its launches, which fail for want of a device: never with one, the addresses
# here are made up.
pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="made-up addresses: only where nothing can be launched")

ADDR = 1 << 20   # 256-byte aligned
ODD = ADDR + 8   # aligned for every element, not as a workspace
BIG = 1 << 40


@pytest.fixture(scope="module")
def gsi():
    from paper_2605_03109_amd import gsi as g

    return g


def _project(gsi, d, k, B, udtype, xdtype, ws, nbytes):
    return gsi.lib.gsi_project(ADDR, ADDR, d, k, B, udtype, xdtype, ADDR, ADDR, ADDR, ADDR, ws, nbytes, None)


def _tables(gsi, d, k, m, dtype):
    inp, mp = (gsi.InputDesc * 1)(), (gsi.MapDesc * 1)()
    for f in ("U", "X", "C", "R", "rnorm", "xnorm", "mask", "fired_idx", "n_fired"):
        setattr(inp[0], f, ADDR)
    inp[0].d, inp[0].k, inp[0].udtype, inp[0].xdtype, inp[0].src_map = d, k, dtype, gsi.GSI_F32, -1
    mp[0].W = mp[0].M = mp[0].Y = ADDR
    mp[0].m, mp[0].wdtype, mp[0].input_id = m, dtype, 0
    return mp, inp


@pytest.mark.parametrize("ws", [None, ODD])
@pytest.mark.parametrize("B", [1, 9, 128])
@pytest.mark.parametrize("k", [24, 200, 264])
def test_no_workspace_at_a_ragged_rank(gsi, k, B, ws):
    """These ranks needed none: memory that cannot be used counts as none, whatever size comes with it."""
    for dtype in (gsi.GSI_F32, gsi.GSI_BF16):
        assert _project(gsi, 1024, k, B, dtype, gsi.GSI_F32, ws, BIG) == gsi.GSI_ERR_HIP, gsi.last_error()
    if B > 1:  # (a single token keeps its tables there); 257 rows have no partial products either
        mp, inp = _tables(gsi, 1024, k, 257, gsi.GSI_BF16)
        assert gsi.lib.gsi_layer_stack(mp, 1, inp, 1, B, 0.05, ws, BIG, None) == gsi.GSI_ERR_HIP, gsi.last_error()
    # where a workspace was needed it still is
    assert _project(gsi, 1024, 64, B, gsi.GSI_BF16, gsi.GSI_F32, ws, BIG) == (
        gsi.GSI_ERR_WORKSPACE if ws is None else gsi.GSI_ERR_ALIGN)


# (d, k, B): the size that gsi_workspace_bytes named while ranks of 8, 16 and 32 columns ran on the FMA kernels
FORMER = {(4096, 32, 64): 147456, (16384, 32, 128): 655360, (65536, 32, 128): 1048576, (16384, 8, 2): 2304}


@pytest.mark.parametrize("shape", sorted(FORMER))
def test_former_sizes_of_small_ranks(gsi, shape):
    d, k, B = shape
    for xdtype in (gsi.GSI_F32, gsi.GSI_BF16):
        assert _project(gsi, d, k, B, gsi.GSI_BF16, xdtype, ADDR, FORMER[shape]) == gsi.GSI_ERR_HIP, gsi.last_error()
        assert _project(gsi, d, k, B, gsi.GSI_BF16, xdtype, ADDR, FORMER[shape] - 256) == gsi.GSI_ERR_WORKSPACE
    assert gsi.workspace_bytes(gsi.CALL_PROJECT, 0, d, k, B) > FORMER[shape]
