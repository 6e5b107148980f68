"""Prefill-sized calls over several inputs and maps: the grouped products against the fp64 oracle and against the
separate calls, at the edges of row tiles, column tiles and 64-token norm groups; the smaller workspace."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

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


def stack_of(gsi, pu, w, flags=()):
    dgs = [pu.DeviceGroup(w, g) for g in w.groups]
    inputs = [{"U": dg.U, "X": dg.X, "flags": flags[i] if i < len(flags) else 0} for i, dg in enumerate(dgs)]
    maps, where = [], []
    for i, (g, dg) in enumerate(zip(w.groups, dgs)):
        for name, _, _ in g.maps:
            maps.append({"W": dg.W[name], "M": dg.M[name], "input_id": i})
            where.append((i, name))
    return dgs, gsi.LayerStack(inputs, maps, w.T, w.eps), where


# one token over a row tile; one short of two; ragged both ways; more tokens than a gate chunk; contractions long enough
# to be split (d, ffn) and ranks of one k-tile
@pytest.mark.parametrize("d,ffn,k,T,rate,xdtype", [(512, 1088, 64, 129, 0.2, "f32"), (768, 2048, 128, 255, 0.0, "bf16"),
                                                   (1024, 4160, 192, 333, 0.3, "f32"), (512, 1024, 64, 1091, 1.0, "bf16")])
def test_block_prefill(gsi, pu, d, ffn, k, T, rate, xdtype):
    w = wl.transformer_block("prefill", d, ffn, k, T, rate, 1.5, 41000 + d + T, xdtype=xdtype)
    print(f"case prefill block d={d} ffn={ffn} k={k} T={T} rate={rate} x {xdtype}", flush=True)
    dgs, st, where = stack_of(gsi, pu, w)
    st.run()
    torch.cuda.synchronize()
    for i, (g, dg) in enumerate(zip(w.groups, dgs)):
        og = pu.OracleGroup(w, g)
        ref = og.run()
        mask = pu.check_projection(st.inputs_t[i], ref, w.eps)
        sep = pu.run_separate_calls(dg, w.eps)
        for key in ("C", "R", "rnorm", "xnorm", "mask", "n_fired"):
            assert torch.equal(st.inputs_t[i][key], sep[key]), key
        for j, (gi, name) in enumerate(where):
            if gi != i:
                continue
            pu.check_outputs(st.maps_t[j]["Y"], og.W[name], og.M[name], gsi.bits_of(dg.M[name]), w.wdtype, ref, mask)
            assert torch.equal(st.maps_t[j]["Y"], sep["Y"][name]), name


def test_mixed_slow_paths_and_dense(gsi, pu):
    """Inputs with and without the W x form in one call: every map as in a call of its own; the dense stack likewise."""
    w = wl.transformer_block("prefill", 512, 1024, 64, 300, 0.25, 1.5, 42000, xdtype="bf16")
    flags = (gsi.INPUT_SLOW_PATH_WX, 0, gsi.INPUT_SLOW_PATH_WX, 0)
    dgs, st, where = stack_of(gsi, pu, w, flags)
    st.run()
    Y = [t["Y"].clone() for t in st.maps_t]
    st.run_dense()
    torch.cuda.synchronize()
    for j, (i, name) in enumerate(where):
        one = gsi.layer_stack([{"U": dgs[i].U, "X": dgs[i].X, "flags": flags[i]}],
                              [{"W": dgs[i].W[name], "M": dgs[i].M[name], "input_id": 0}], w.T, w.eps)
        torch.cuda.synchronize()
        assert torch.equal(Y[j], one.maps_t[0]["Y"]), name
        dense = gsi.dense_linear(dgs[i].W[name], dgs[i].X)
        assert torch.equal(st.maps_t[j]["Y"], dense), name
        if flags[i]:
            fired = st.inputs_t[i]["mask"].bool()
            assert pu.rel_l2_rows(Y[j][fired].cpu().double().numpy(), dense[fired].cpu().double().numpy()).max() <= 2e-6


def test_smaller_workspace_is_served(gsi, pu):
    """A call that brings less than the query names, but what calls of its shape once asked for."""
    w = wl.tiny(16384, 64, 264, 140, 30, seed=43000, wdtype="bf16")  # a long contraction: more splits than there once were
    dgs, st, where = stack_of(gsi, pu, w)
    st.run()
    torch.cuda.synchronize()
    args = (st._mp, len(st.maps_t), st._in, len(st.inputs_t), w.T)
    need = int(gsi.lib.gsi_layer_stack_workspace_bytes(*args))
    s = torch.cuda.current_stream().cuda_stream
    rc = gsi.lib.gsi_layer_stack(*args, w.eps, st.ws.data_ptr(), need - 256, s)
    torch.cuda.synchronize()
    assert rc == gsi.GSI_OK, gsi.last_error()
    # sums split differently, and r, once rounded to bf16 for its product, may round to the other neighbour: the oracle's bars
    og = pu.OracleGroup(w, w.groups[0])
    ref = og.run()
    mask = pu.check_projection(st.inputs_t[0], ref, w.eps)
    pu.check_outputs(st.maps_t[0]["Y"], og.W["w"], og.M["w"], gsi.bits_of(dgs[0].M["w"]), w.wdtype, ref, mask)
    assert gsi.lib.gsi_layer_stack(*args, w.eps, st.ws.data_ptr(), 4096, s) == gsi.GSI_ERR_WORKSPACE
