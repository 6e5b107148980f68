"""Ranks that are not a power of two of 16-byte pieces, and bf16 activations in decode batches: the vector and
matrix-core kernels against the fp64 oracle, at the edges of lanes, MFMA steps and column blocks."""
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


# one piece, 3, 25, 33, 63 of 64 pieces; one column past and short of a 64-column block and a 32-column step; ragged
# slabs (d = 1160 is no multiple of the slab sizes, and no multiple of 128: the vector kernels take its batches)
@pytest.mark.parametrize("d,k,m,T,nf,wdtype,xdtype", [
    (1024, 24, 264, 5, 2, "bf16", "f32"), (2048, 200, 520, 7, 2, "bf16", "bf16"), (2176, 264, 300, 33, 9, "bf16", "f32"),
    (2560, 504, 260, 18, 18, "bf16", "bf16"), (1024, 72, 512, 128, 40, "bf16", "f32"), (1024, 56, 36, 2, 0, "bf16", "bf16"),
    (1160, 200, 264, 6, 3, "bf16", "bf16"), (1160, 136, 264, 6, 3, "f32", "f32"), (768, 44, 300, 5, 2, "f32", "f32"),
    (4096, 192, 1032, 64, 10, "bf16", "bf16"), (20480, 200, 136, 5, 2, "bf16", "bf16"),
    (1024, 128, 260, 23, 6, "bf16", "bf16"), (1024, 8, 260, 9, 2, "bf16", "f32")])
def test_ragged_ranks_and_bf16_batches(gsi, pu, d, k, m, T, nf, wdtype, xdtype):
    w = wl.tiny(d, k, m, T, nf, seed=31000 + d + k + m, wdtype=wdtype, xdtype=xdtype)
    print(f"case ragged d={d} k={k} m={m} T={T} nf={nf} {wdtype} x {xdtype}", flush=True)
    g = w.groups[0]
    dg = pu.DeviceGroup(w, g)
    worst = pu.check_group(w, g, [(0, T), (0, 1), (T - 1, T), (0, min(T, 2))], dg)
    print(f"  worst rel-L2 {worst:.3e}", flush=True)
    # the whole call: the bits of the separate ones; W x form: a fired token equals the dense product to rounding
    sep = pu.run_separate_calls(dg, w.eps)
    inp, mp = {"U": dg.U, "X": dg.X}, {"W": dg.W["w"], "M": dg.M["w"], "input_id": 0}
    st = gsi.layer_stack([inp], [mp], T, w.eps)
    wx = gsi.layer_stack([dict(inp, flags=gsi.INPUT_SLOW_PATH_WX)], [mp], T, w.eps)
    torch.cuda.synchronize()
    for key in ("C", "R", "rnorm", "xnorm", "mask", "n_fired"):
        assert torch.equal(st.inputs_t[0][key], sep[key]), key
    assert torch.equal(st.maps_t[0]["Y"], sep["Y"]["w"])
    mask = sep["mask"].bool().cpu().numpy()
    og = pu.OracleGroup(w, g)
    dense = O.dense_linear(og.W["w"], og.X)
    bar = 2e-5 if wdtype == "bf16" else 1e-5
    if mask.any():
        assert pu.rel_l2_rows(wx.maps_t[0]["Y"].cpu().numpy().astype(np.float64)[mask], dense[mask]).max() <= bar
    Yd = gsi.dense_linear(dg.W["w"], dg.X).cpu().numpy().astype(np.float64)
    assert pu.rel_l2_rows(Yd, dense).max() <= bar


@pytest.mark.parametrize("d,k,B", [(1024, 200, 1), (1024, 200, 9)])
def test_ragged_rank_without_workspace(gsi, pu, d, k, B):
    """A caller that brings no workspace for such a rank is served by the generic kernels, as ever."""
    w = wl.tiny(d, k, 264, B, 0, seed=32000 + B, wdtype="bf16")
    dg, og = pu.DeviceGroup(w, w.groups[0]), pu.OracleGroup(w, w.groups[0])
    C, R, rn, xn = [torch.empty(s, device="cuda") for s in ((B, k), (B, d), (B,), (B,))]
    s = torch.cuda.current_stream().cuda_stream
    rc = gsi.lib.gsi_project(dg.U.data_ptr(), dg.X.data_ptr(), d, k, B, 1, 0, C.data_ptr(), R.data_ptr(), rn.data_ptr(),
                             xn.data_ptr(), None, 0, s)
    torch.cuda.synchronize()
    assert rc == gsi.GSI_OK, gsi.last_error()
    assert pu.rel_l2_rows(C.cpu().numpy().astype(np.float64), og.run()["C"]).max() <= 1e-5


def test_infinite_and_nan_activations_stay_in_their_token(gsi, pu):
    d, k, T = 1024, 200, 20
    w = wl.tiny(d, k, 264, T, 4, seed=33000, wdtype="bf16", xdtype="bf16")
    dg = pu.DeviceGroup(w, w.groups[0])
    clean = pu.run_separate_calls(dg, w.eps)
    dg.X = dg.X.clone()
    dg.X[3, 17], dg.X[11, 5] = float("inf"), float("nan")
    res = pu.run_separate_calls(dg, w.eps)
    torch.cuda.synchronize()
    keep = [t for t in range(T) if t not in (3, 11)]
    for key in ("C", "R", "rnorm", "xnorm"):
        assert torch.equal(res[key][keep], clean[key][keep]), key
    u = dg.U[17].float()
    assert torch.equal(res["C"][3][u != 0], (torch.sign(u) * float("inf"))[u != 0])  # one infinite term: c is infinite
    assert torch.isnan(res["C"][11]).all() and torch.isinf(res["xnorm"][3]) and torch.isnan(res["xnorm"][11])


@pytest.mark.parametrize("d,m", [(768, 3072), (2048, 8192), (2080, 512), (2048, 8196)])
def test_dense_products_of_two_bf16_tokens(gsi, pu, d, m):
    """Both sides of the rule that gives short rows to the FMA kernel; a stack of both kinds equals its separate products."""
    g = torch.Generator(device="cuda").manual_seed(d + m)
    X = torch.randn(2, d, generator=g, device="cuda").to(torch.bfloat16)
    Ws = [(torch.randn(r, d, generator=g, device="cuda") / d**0.5).to(torch.bfloat16) for r in (m, 64, 8200)]
    st = gsi.LayerStack([{"U": torch.zeros(d, 64, dtype=torch.bfloat16, device="cuda"), "X": X}],
                        [{"W": W, "M": torch.zeros(W.shape[0], 64, dtype=torch.bfloat16, device="cuda"), "input_id": 0} for W in Ws],
                        2, 0.1)
    st.run_dense()
    torch.cuda.synchronize()
    for W, t in zip(Ws, st.maps_t):
        ref = X.double() @ W.double().T
        assert pu.rel_l2_rows(t["Y"].cpu().double().numpy(), ref.cpu().numpy()).max() <= 1e-6
        assert torch.equal(t["Y"], gsi.dense_linear(W, X))
