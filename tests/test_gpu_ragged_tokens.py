"""One-token stacks at ranks that are not a power of two of 16-byte pieces: few inputs, more than one launch's arguments
describe, the single-pass gate (which such a rank answers with the explicit one), and images kept as E4M3 codes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle.gsi_oracle as O  # noqa: E402
from paper_2605_03109_amd import workload as wl  # noqa: E402

T = 5


@pytest.fixture(scope="module")
def gsi():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_03109_amd import gsi as g

    return g


@pytest.fixture(scope="module")
def pu(gsi):
    import parity_util

    return parity_util


def _run(st):
    for t in range(T):
        st.refresh(token_offset=t, B=1)
        st.run()
    torch.cuda.synchronize()
    return ([{key: ti[key].clone() for key in ("C", "R", "rnorm", "xnorm", "mask")} for ti in st.inputs_t],
            [mt["Y"].clone() for mt in st.maps_t])


# 4 inputs: arguments of the launches; 17: descriptor tables.  25 and 13 of 32 pieces; rows with a tail in every slab size
@pytest.mark.parametrize("n,d,k,wdtype,xdtype", [(1, 2048, 200, "bf16", "f32"), (4, 1160, 104, "bf16", "bf16"),
                                                 (4, 516, 100, "f32", "f32"), (17, 1160, 200, "bf16", "f32"),
                                                 (17, 516, 44, "f32", "f32")])
def test_one_token_stack(gsi, pu, n, d, k, wdtype, xdtype):
    print(f"case ragged token stack: {n} inputs d={d} k={k} {wdtype} x {xdtype}", flush=True)
    ws = [wl.tiny(d, k, 260 + 8 * i, T, 2, seed=71000 + 100 * n + i, wdtype=wdtype, xdtype=xdtype) for i in range(n)]
    dgs = [pu.DeviceGroup(w, w.groups[0]) for w in ws]
    inputs = [{"U": dg.U, "X": dg.X} for dg in dgs]
    maps = [{"W": dg.W["w"], "M": dg.M["w"], "input_id": i} for i, dg in enumerate(dgs)]
    st = gsi.LayerStack(inputs, maps, T, ws[0].eps)
    st.refresh(token_offset=0, B=1)
    st.ws.fill_(0xFF)
    ins, ys = _run(st)
    again = _run(st)
    single = _run(gsi.LayerStack([dict(i, flags=gsi.INPUT_GATE_SINGLE_PASS, gram=gsi.build_gram(i["U"])) for i in inputs],
                                 maps, T, ws[0].eps))
    for other in (again, single):
        for a, b in zip(ins, other[0]):
            for key in a:
                assert torch.equal(a[key], b[key]), key
        assert all(torch.equal(a, b) for a, b in zip(ys, other[1]))
    for w, dg, ti, y in zip(ws, dgs, ins, ys):
        og = pu.OracleGroup(w, w.groups[0])
        ref = og.run()
        m = ti["mask"].cpu().numpy()
        assert np.array_equal(m.astype(bool), w.groups[0].fired_design)
        res = dict(ti, n_fired=torch.tensor([int(m.sum())], dtype=torch.int32),
                   fired_idx=torch.from_numpy(np.nonzero(m)[0].astype(np.int32)))
        pu.check_projection(res, ref, w.eps)
        pu.check_outputs(y, og.W["w"], og.M["w"], gsi.bits_of(dg.M["w"]), wdtype, ref, m)


# 3, 6 and 13 pieces of 16 codes: below and above half a wave's row, and two odd counts
@pytest.mark.parametrize("k", [48, 96, 208])
@pytest.mark.parametrize("wx", [False, True])
def test_codes_equal_their_expansion(gsi, pu, k, wx):
    """The image as E4M3 codes and the same values as bf16: one oracle, 2e-5 for the fp32 sums of either."""
    d, m = 1160, 264
    print(f"case ragged codes k={k} wx={wx}", flush=True)
    w = wl.tiny(d, k, m, T, 2, seed=72000 + k, wdtype="bf16")
    dg, og = pu.DeviceGroup(w, w.groups[0]), pu.OracleGroup(w, w.groups[0])
    ref = og.run()
    M8, scale = gsi.quantize_image_fp8(dg.M["w"])
    Mdeq = O.dequantize_image_fp8(M8.cpu().numpy(), scale.cpu().numpy())
    inp = {"U": dg.U, "X": dg.X, "flags": gsi.INPUT_SLOW_PATH_WX if wx else 0}
    for mp in ({"M": M8, "M_scale": scale}, {"M": gsi.to_device(wl.f32_to_bf16_bits(Mdeq.astype(np.float32)), "bf16")}):
        ins, ys = _run(gsi.LayerStack([inp], [dict(mp, W=dg.W["w"], input_id=0)], T, w.eps))
        mask = ins[0]["mask"].cpu().numpy()
        assert np.array_equal(mask.astype(bool), w.groups[0].fired_design)
        want = (O.gated_linear_alg1(og.W["w"], Mdeq, ref["C"], og.X, mask) if wx
                else O.gated_linear(og.W["w"], Mdeq, ref["C"], ref["R"], mask))
        assert pu.rel_l2_rows(ys[0].cpu().double().numpy(), want).max() <= 2e-5
