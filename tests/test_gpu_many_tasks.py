"""One token through stacks of more inputs and maps than a wave has lanes: the launches over descriptor tables look a workgroup's
task up in two steps there.  Unlike sizes throughout, so that a wrong task shows as wrong or unwritten results."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SENTINEL = 7.25
EPS = 0.3


# one step (up to 64), the first counts of two and three entries a group, last groups shorter than the others
@pytest.mark.parametrize("n_in,n_maps", [(17, 64), (64, 65), (65, 127), (20, 128), (129, 129), (66, 193), (193, 130), (3, 193)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_many_inputs_and_maps(n_in, n_maps, dtype):
    from paper_2605_03109_amd import gsi

    print(f"case many tasks inputs={n_in} maps={n_maps} {dtype}", flush=True)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    g = torch.Generator(device="cuda").manual_seed(1000 * n_in + n_maps)
    dims, ranks, rows = (128, 520, 1024, 2056, 192), (16, 64, 8, 128, 32, 8, 64), (1, 130, 7, 300, 33, 64, 5, 17, 4, 259, 3)
    inputs, maps = [], []
    for i in range(n_in):
        d, k = dims[i % len(dims)], ranks[i % len(ranks)]
        U = torch.linalg.qr(torch.randn(d, k, generator=g, device="cuda", dtype=torch.float64))[0].to(dt).contiguous()
        x = torch.randn(1, d, generator=g, device="cuda")
        if i % 3:  # two of three tokens lie in the subspace but for a twentieth
            inside = (x.double() @ U.double()) @ U.double().T
            x = (inside / inside.norm() + 0.05 * x.double() / x.norm()).float()
        inputs.append({"U": U, "X": x, "gram": gsi.build_gram(U),
                       "flags": gsi.INPUT_GATE_SINGLE_PASS | (gsi.INPUT_SLOW_PATH_WX if i % 4 == 0 else 0)})
    for j in range(n_maps):
        i = j * 7 % n_in  # (no order of the maps by input; every input has one if there are as many)
        U, m = inputs[i]["U"], rows[j % len(rows)]
        W = (torch.randn(m, U.shape[0], generator=g, device="cuda") / U.shape[0]**0.5).to(dt)
        maps.append({"W": W, "M": (W.double() @ U.double()).to(dt), "input_id": i})
    mapped = {mp["input_id"] for mp in maps}  # (an input without a map may have its r written)
    st = gsi.LayerStack(inputs, maps, 1, EPS)

    def clear():
        for t in st.inputs_t:
            for name in ("C", "R", "rnorm", "xnorm"):
                t[name].fill_(SENTINEL)
            t["mask"].fill_(9)
            t["n_fired"].fill_(9)
        for t in st.maps_t:
            t["Y"].fill_(SENTINEL)
        st.ws.fill_(0xFF)
        torch.cuda.synchronize()

    refs = []
    for t in st.inputs_t:
        x, U = t["X"].double(), t["U"].double()
        c = x @ U
        r = x - c @ U.T
        rho = float(r.norm() / x.norm())
        assert abs(rho - EPS) > 0.02
        refs.append((x, c, r, rho >= EPS))
    fired = [f for _, _, _, f in refs]
    assert any(fired) and not all(fired)

    def check():
        rel = lambda a, b: float(torch.linalg.norm(a.double() - b) / torch.linalg.norm(b))
        for i, (t, (x, c, r, f)) in enumerate(zip(st.inputs_t, refs)):
            d, k = t["U"].shape
            # fp32 sums of d (c) and k (r) terms: random-walk growth of roundings of 2^-24, four times that; r against x
            assert rel(t["C"], c) <= 4 * 2**-24 * d**0.5, i
            assert bool(t["mask"]) == f and int(t["n_fired"]) == int(f), i
            assert abs(float(t["xnorm"]) / float(x.norm()) - 1) <= 2**-22, i
            if f and not t["flags"] & gsi.INPUT_SLOW_PATH_WX:
                assert float((t["R"].double() - r).norm() / x.norm()) <= 4 * 2**-24 * (d**0.5 + k**0.5), i
            elif i in mapped:
                assert bool((t["R"] == SENTINEL).all()), i
        for j, t in enumerate(st.maps_t):
            inp, (x, c, r, f) = st.inputs_t[t["input_id"]], refs[t["input_id"]]
            d, k = inp["U"].shape
            W, M = t["W"].double(), t["M"].double()
            wx = inp["flags"] & gsi.INPUT_SLOW_PATH_WX
            y = x @ W.T if f and wx else c @ M.T + r @ W.T if f else c @ M.T
            # against the length of what enters: a map of one row may cancel to nothing
            scale = float(x.norm()) * float(W.norm() + M.norm())
            assert float((t["Y"].double() - y).norm()) <= 4 * 2**-24 * (d**0.5 + k**0.5) * scale, j

    clear()
    st.run()
    torch.cuda.synchronize()
    check()
    if len(mapped) < n_in:
        return  # (a plan takes no input without a map)
    clear()
    plan, mem = st.build_plan()
    for _ in range(2):
        st.run_plan(plan)
        torch.cuda.synchronize()
        check()
