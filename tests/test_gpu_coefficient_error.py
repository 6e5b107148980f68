"""One token: cutting the columns of a basis costs no precision: the error of c against that of whole rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _whole_rows(U, x, rows, groups):
    """c in fp32 as whole rows give it: slabs of `rows` rows, dealt to `groups` row groups that are added in order, then the slabs.
    A product of fp32 and a sum are formed in 64 bits and rounded once, as an fma does."""
    d, k = U.shape
    slabs = d // rows
    acc = np.zeros((slabs, groups, k), np.float32)
    u = U.astype(np.float64).reshape(slabs, rows // groups, groups, k)
    xs = x.astype(np.float64).reshape(slabs, rows // groups, groups, 1)
    for i in range(rows // groups):
        acc = (u[:, i] * xs[:, i] + acc.astype(np.float64)).astype(np.float32)
    part = np.zeros((slabs, k), np.float32)
    for g in range(groups):
        part += acc[:, g]
    c = np.zeros(k, np.float32)
    for s in range(slabs):
        c += part[s]
    return c


# ranks in four blocks, evenly and raggedly; two blocks; fp32; one block (the same groups of rows on both sides)
@pytest.mark.parametrize("d,k,dtype,groups", [
    (4096, 200, "bf16", 8), (4096, 256, "bf16", 8), (4096, 512, "bf16", 4), (4096, 128, "bf16", 16), (2048, 256, "f32", 4),
    (4096, 64, "bf16", 32)])
def test_error_of_coefficients(d, k, dtype, groups):
    from paper_2605_03109_amd import gsi

    print(f"case coefficient error d={d} k={k} {dtype}", flush=True)
    tokens = 24
    rows = max(d // 32, 8 * groups)
    g = torch.Generator(device="cuda").manual_seed(d + k)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    U = (torch.randn(d, k, generator=g, device="cuda") / d**0.5).to(dt)
    X = torch.randn(tokens, d, generator=g, device="cuda")
    exact = (X.double() @ U.double()).cpu().numpy()
    C = torch.cat([gsi.project(U, X[t:t + 1])[0] for t in range(tokens)]).cpu().numpy()
    u, x = U.float().cpu().numpy(), X.cpu().numpy()
    whole = np.stack([_whole_rows(u, x[t], rows, groups) for t in range(tokens)])
    err, ref = np.linalg.norm(C - exact), np.linalg.norm(whole - exact)
    # both are root mean squares of tokens * k >= 1500 independent errors: 4 % of chance at two standard deviations
    print(f"  error {err:.3e}, whole rows {ref:.3e}, ratio {err / ref:.3f}", flush=True)
    assert err <= 1.04 * ref, (err, ref)
