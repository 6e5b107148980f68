"""Decode batches that bring exactly the workspace that the query named while ranks of 8, 16 and 32 columns ran on the FMA
kernels: served by those kernels, to the oracle's bars."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2605_03109_amd import workload as wl  # noqa: E402


@pytest.mark.parametrize("d,k,T,former,xdtype", [(1024, 16, 9, 2560, "f32"), (1024, 32, 40, 23040, "bf16"),
                                                 (16384, 8, 2, 2304, "f32")])
def test_small_rank_with_the_former_workspace(d, k, T, former, xdtype):
    import parity_util as pu
    from paper_2605_03109_amd import gsi

    w = wl.tiny(d, k, 64, T, 1, seed=53000 + d + k, wdtype="bf16", xdtype=xdtype)
    print(f"case former workspace d={d} k={k} T={T} x {xdtype}", flush=True)
    dg, og = pu.DeviceGroup(w, w.groups[0]), pu.OracleGroup(w, w.groups[0])
    ws = torch.empty(former, dtype=torch.uint8, device="cuda")
    C, R, rn, xn = out = [torch.empty(s, device="cuda") for s in ((T, k), (T, d), (T,), (T,))]
    call = lambda n: gsi.lib.gsi_project(dg.U.data_ptr(), dg.X.data_ptr(), d, k, T, gsi.GSI_BF16, gsi.dtype_code(dg.X),
                                         *[o.data_ptr() for o in out], ws.data_ptr(), n,
                                         torch.cuda.current_stream().cuda_stream)
    assert call(former - 256) == gsi.GSI_ERR_WORKSPACE
    assert call(former) == gsi.GSI_OK, gsi.last_error()
    torch.cuda.synchronize()
    ref = og.run()
    host = lambda t: t.cpu().numpy().astype(np.float64)
    # fp32 sums of d terms: the bars of the other projection tests
    assert pu.rel_l2_rows(host(C), ref["C"]).max() <= 1e-5
    assert np.abs(host(R) - ref["R"]).max() <= 1e-5 * np.abs(og.X).max()
    assert np.abs(host(rn) - ref["rnorm"]).max() <= 1e-5 * ref["xnorm"].max()
    assert np.abs(host(xn) - ref["xnorm"]).max() <= 1e-5 * ref["xnorm"].max()
