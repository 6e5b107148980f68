"""Decode batches with fp32 storage on the fp32 matrix instructions: token tiles and groups, row and column tails, every
fired count, bf16 activations, the W x form, the dense product, and the smaller workspace."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle.gsi_oracle as O  # noqa: E402
from paper_2605_03109_amd import workload as wl  # noqa: E402


@pytest.fixture(scope="module")
def gsi():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_03109_amd import gsi as g

    return g


@pytest.fixture(scope="module")
def pu(gsi):
    import parity_util

    return parity_util


# one tile and one token over it; a group of four tiles and one over; the whole call; rows 1 and 15 past a 16-row block;
# contractions of 4 and 36 columns past a piece; slabs with a ragged end
@pytest.mark.parametrize("d,k,m,T,nf,xdtype", [(768, 64, 3072, 16, 4, "f32"), (516, 36, 257, 17, 17, "f32"),
                                               (1044, 68, 303, 64, 1, "bf16"), (640, 256, 97, 65, 64, "f32"),
                                               (4100, 128, 130, 128, 128, "bf16"), (256, 4, 16, 2, 0, "f32")])
def test_f32_batches(gsi, pu, d, k, m, T, nf, xdtype):
    w = wl.tiny(d, k, m, T, nf, seed=51000 + d + k + m, wdtype="f32", xdtype=xdtype)
    print(f"case f32 batch d={d} k={k} m={m} T={T} nf={nf} x {xdtype}", flush=True)
    g = w.groups[0]
    dg, og = pu.DeviceGroup(w, g), pu.OracleGroup(w, g)
    worst = pu.check_group(w, g, [(0, T), (0, min(T, 3))], dg, og)
    print(f"  worst rel-L2 {worst:.3e}", flush=True)
    sep = pu.run_separate_calls(dg, w.eps)
    inp, mp = {"U": dg.U, "X": dg.X}, {"W": dg.W["w"], "M": dg.M["w"], "input_id": 0}
    st = gsi.layer_stack([inp], [mp], T, w.eps)
    wx = gsi.layer_stack([dict(inp, flags=gsi.INPUT_SLOW_PATH_WX)], [mp], T, w.eps)
    torch.cuda.synchronize()
    for key in ("C", "R", "rnorm", "xnorm", "mask", "n_fired"):
        assert torch.equal(st.inputs_t[0][key], sep[key]), key
    assert torch.equal(st.maps_t[0]["Y"], sep["Y"]["w"])
    dense = gsi.dense_linear(dg.W["w"], dg.X)
    mask = sep["mask"].bool()
    if mask.any():  # the same sums in the same order
        assert torch.equal(wx.maps_t[0]["Y"][mask], dense[mask])
    assert pu.rel_l2_rows(dense.cpu().double().numpy(), O.dense_linear(og.W["w"], og.X)).max() <= 1e-5


def test_f32_batch_with_the_smaller_workspace(gsi, pu):
    """A call that brings less than the query names, but what calls of its shape once asked for, takes the FMA kernels;
    one step less was refused and is."""
    d, k, m, T, full, former = 768, 64, 300, 16, 26368, 26112
    w = wl.tiny(d, k, m, T, 4, seed=52000, wdtype="f32")
    dg, og = pu.DeviceGroup(w, w.groups[0]), pu.OracleGroup(w, w.groups[0])
    assert gsi.workspace_bytes(gsi.CALL_PROJECT, 0, d, k, T) == full
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    out = [torch.empty(s, device="cuda") for s in ((T, k), (T, d), (T,), (T,))]
    s = torch.cuda.current_stream().cuda_stream

    def call(nbytes):
        return gsi.lib.gsi_project(dg.U.data_ptr(), dg.X.data_ptr(), d, k, T, 0, 0, *[o.data_ptr() for o in out],
                                   ws.data_ptr(), nbytes, s)

    assert call(former - 256) == gsi.GSI_ERR_WORKSPACE
    assert call(former) == gsi.GSI_OK, gsi.last_error()
    torch.cuda.synchronize()
    ref = og.run()
    assert pu.rel_l2_rows(out[0].cpu().double().numpy(), ref["C"]).max() <= 1e-5
    assert np.abs(out[2].cpu().double().numpy() - ref["rnorm"]).max() <= 1e-5 * ref["xnorm"].max()
