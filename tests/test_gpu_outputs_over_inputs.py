"""Outputs that lie over activations of the same call: every x is read before it is overwritten, whatever launches the
images and the weight terms of a call share.  The bits are those of the call with buffers of its own."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _data(n, d, k, T, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    out = []
    for _ in range(n):
        U = torch.linalg.qr(r(d, k).double())[0].to(torch.bfloat16).contiguous()
        noise = 0.3 * k**0.5 * torch.rand(T, 1, generator=g, device="cuda")  # 0 .. 0.3 of the part inside the basis
        X = (r(T, k) @ U.float().T + noise * r(T, d) / d**0.5).contiguous()
        Ws = [(r(m, d) / d**0.5).to(torch.bfloat16) for m in (d // 2 + 4, d)]
        out.append((U, X, Ws, [(W.float() @ U.float()).to(torch.bfloat16) for W in Ws]))
    return out


def _stack(gsi, data, T, wx, gate, over):
    """over: inputs i whose second map writes to the X of input i + 1 (the last one: of the first)."""
    n, xs = len(data), [X.clone() for _, X, _, _ in data]
    inputs, maps = [], []
    for i, (U, _, Ws, Ms) in enumerate(data):
        flags = (gsi.INPUT_SLOW_PATH_WX if wx and i % 2 else 0) | (gsi.INPUT_GATE_SINGLE_PASS if gate == "single" else 0)
        inputs.append({"U": U, "X": xs[i], "flags": flags, "gram": gsi.build_gram(U) if gate == "single" else None})
        maps += [{"W": Ws[0], "M": Ms[0], "input_id": i},
                 {"W": Ws[1], "M": Ms[1], "input_id": i, "Y": xs[(i + 1) % n] if i in over else None}]
    return gsi.LayerStack(inputs, maps, T, 0.15)


# one set of inputs, several sets, the table launches; a token, the FMA and matrix-core batches, a prefill
@pytest.mark.parametrize("wx", [False, True])
@pytest.mark.parametrize("n,d,k,T,gate", [(2, 1024, 64, 1, "explicit"), (2, 1024, 200, 1, "explicit"), (2, 1024, 64, 1, "single"),
                                          (18, 512, 64, 1, "explicit"), (18, 512, 72, 1, "explicit"), (18, 512, 64, 1, "single"),
                                          (2, 1024, 64, 9, "explicit"), (2, 1024, 200, 40, "explicit"), (18, 512, 64, 33, "explicit"),
                                          (2, 1024, 64, 140, "explicit"), (6, 512, 128, 300, "explicit")])
def test_outputs_over_the_next_input(n, d, k, T, gate, wx):
    from paper_2605_03109_amd import gsi

    print(f"case outputs over inputs n={n} d={d} k={k} T={T} {gate} wx={wx}", flush=True)
    data = _data(n, d, k, T, 1000 * n + k + T)
    want, have = (_stack(gsi, data, T, wx, gate, over) for over in ((), range(n)))
    want.run()
    have.run()
    torch.cuda.synchronize()
    for a, b in zip(want.inputs_t, have.inputs_t):
        for key in ("C", "R", "rnorm", "xnorm", "mask", "fired_idx", "n_fired"):
            assert torch.equal(a[key], b[key]), key
    for j, (a, b) in enumerate(zip(want.maps_t, have.maps_t)):
        assert torch.equal(a["Y"], b["Y"]), j
    assert 0 < sum(int(t["n_fired"]) for t in want.inputs_t) < n * T or n * T < 4


@pytest.mark.parametrize("T", [1, 40, 140])
def test_dense_output_over_another_input(T):
    from paper_2605_03109_amd import gsi

    data = _data(3, 512, 64, T, T)
    want, have = (_stack(gsi, data, T, False, "explicit", over) for over in ((), (0,)))
    want.run_dense()
    have.run_dense()
    torch.cuda.synchronize()
    for j, (a, b) in enumerate(zip(want.maps_t, have.maps_t)):
        assert torch.equal(a["Y"], b["Y"]), j
