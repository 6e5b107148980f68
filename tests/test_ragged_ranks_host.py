"""Host-side rules for ranks that are not a power of two of 16-byte pieces: workspace queries and what stays refused."""
import ctypes

import pytest

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gsi():
    from paper_2605_03109_amd import gsi as g

    return g


@pytest.mark.parametrize("k", [24, 72, 200, 504])
def test_workspace_query_covers_every_rank(gsi, k):
    for B in (1, 2, 33, 128):
        assert gsi.workspace_bytes(gsi.CALL_PROJECT, 0, 4096, k, B) > 0
    assert gsi.workspace_bytes(gsi.CALL_PROJECT, 0, 4096, 515, 1) == 0  # generic kernels


def test_plan_still_refuses_other_ranks(gsi):
    one = 1 << 20  # an aligned address that is never dereferenced: the call is refused on the host
    inp, mp = (gsi.InputDesc * 1)(), (gsi.MapDesc * 1)()
    i, m = inp[0], mp[0]
    i.U = i.X = i.C = i.R = i.rnorm = i.xnorm = i.mask = i.fired_idx = i.n_fired = i.gram = one
    i.d, i.k, i.udtype, i.xdtype, i.src_map, i.flags = 1024, 200, gsi.GSI_BF16, gsi.GSI_F32, -1, gsi.INPUT_GATE_SINGLE_PASS
    m.W = m.M = m.Y = one
    m.m, m.wdtype, m.input_id = 264, gsi.GSI_BF16, 0
    plan = gsi.StackPlan()
    rc = gsi.lib.gsi_stack_plan_build(mp, 1, inp, 1, one, 1 << 30, one, 1 << 20, ctypes.byref(plan), None)
    assert rc == gsi.GSI_ERR_SHAPE and "planned" in gsi.last_error()
