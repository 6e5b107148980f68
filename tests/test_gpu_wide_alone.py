"""W r of many tokens on tiles whose height follows the launch: a map by itself, in its own call and in a stack, and beside other maps has
the same bits, and those of its 64-bit sums to rounding."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# contractions in parts and in one, column tiles by the eight and ragged; counts of one, of whole fragments of 16 rows and one more, of one tile
# of 256 rows and one more, of all
@pytest.mark.parametrize("d,m,B", [(2112, 2308, 1000), (2176, 7168, 1100), (4096, 4096, 1300)])
@pytest.mark.parametrize("fired", [1, 16, 17, 130, 256, 257, 330, 1000])
def test_alone_and_beside(d, m, B, fired):
    from paper_2605_03109_amd import gsi

    k = 64
    g = torch.Generator(device="cuda").manual_seed(d + m + B)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    U = torch.linalg.qr(r(d, k)).Q.to(torch.bfloat16).contiguous()
    X = r(B, k) @ U.float().T
    X[torch.randperm(B, generator=g, device="cuda")[:fired]] += 0.5 * r(fired, d)
    maps = []
    for n in (m, 4096, 1024, 4100):
        W = (r(n, d) / d**0.5).to(torch.bfloat16)
        maps.append({"W": W, "M": (W.float() @ U.float()).to(torch.bfloat16), "input_id": 0})
    print(f"case alone and beside d={d} m={m} B={B} fired={fired}", flush=True)
    alone, beside = (gsi.LayerStack([{"U": U, "X": X}], q, B, 0.1) for q in (maps[:1], maps))
    alone.run()
    beside.run()
    t, Y = beside.inputs_t[0], beside.maps_t[0]["Y"]
    one = gsi.gated_linear(maps[0]["W"], maps[0]["M"], t["C"], t["R"], t["fired_idx"], t["n_fired"])
    torch.cuda.synchronize()
    assert int(t["n_fired"][0]) == fired
    assert torch.equal(alone.maps_t[0]["Y"], Y) and torch.equal(one, Y)
    C, R, W, M = t["C"].double(), t["R"].double(), maps[0]["W"].double(), maps[0]["M"].double()
    want = C @ M.T
    rows = t["fired_idx"][:fired].long()
    want[rows] += t["R"][rows].to(torch.bfloat16).double() @ W.T
    # 32-bit sums of d exact products, and of k products of operands of 16 mantissa bits: 2^-16 of the norms that bound them
    bar = 2.0**-16 * (C.norm(dim=1).max() * M.norm(dim=1).max() + R.norm(dim=1).max() * W.norm(dim=1).max())
    assert (Y.double() - want).abs().max() <= bar
