"""The work a program has this library do, as measurable cases: gated layer calls from one token to a prefill batch,
the one-time preparation of a block, and the extension of a basis.

Inputs are synthetic: weights N(0, 1/d), orthonormal bases, activations with a decaying spectrum inside the basis and
a residual part whose share of the norm puts each token clearly on one side of the gate's threshold.  Everything is
made on the GPU from the seed; which tokens (or, for one token, which inputs) fire is counted, so that every seed
does the same work.  Images, E4M3 codes and E = U^T U - I are made here with torch, so that a case measures only the
entry points it calls.
"""
import math

import torch

from paper_2605_03109_amd import gsi

EPS = 0.05          # gate threshold of the paper's operating point
DEV = "cuda"
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"bf16": 2, "f32": 4}

# shape of a call: inputs (width) and the maps that read each; "d" and "ffn" are the case's widths
SHAPES = {
    "block": [("d", ["d", "d", "d"]), ("d", ["d"]), ("d", ["ffn"]), ("ffn", ["d"])],  # q k v | o | fc_in | fc_out
    "pair": [("d", ["ffn"]), ("ffn", ["d"])],                                         # fc_in | fc_out
    "one": [("d", ["ffn"])],                                                          # one map, ffn rows
}


def _stack(name, shape, d, ffn, k, tokens, fired, layers=1, w="bf16", x="f32", gate="explicit", slow="mc_wr",
           image="same", call="run"):
    """fired: tokens of a batch that fire, per input; for one token, every fired-th input fires (0: none)."""
    return {"name": name, "kind": "stack", "shape": shape, "d": d, "ffn": ffn, "k": k, "tokens": tokens, "fired": fired,
            "layers": layers, "w": w, "x": x, "gate": gate, "slow": slow, "image": image, "call": call}


def listed():
    return [
        # the smallest call: the MLP up-projection of a small fp32 model, one token that fires, step by step
        _stack("mlp_up_f32_token", "one", 768, 3072, 64, 1, 1, w="f32", call="separate"),
        # one block, one token of a decode loop; at rank 256 almost every token stays on the fast path
        _stack("block_token", "block", 4096, 16384, 256, 1, 0),
        # the same block at a rank that an energy threshold chose
        _stack("block_token_rank200", "block", 4096, 16384, 200, 1, 0),
        # a whole 32-layer model per token, marshalled once; 5 % of the inputs fire
        _stack("model_token_plan", "block", 4096, 16384, 256, 1, 21, layers=32, gate="single", call="plan"),
        # part of a model with 8-bit images and the merged dispatch (a fired token is W x)
        _stack("layers8_token_fp8", "block", 4096, 16384, 128, 1, 21, layers=8, gate="single", slow="wx", image="fp8"),
        # decode batches of a serving loop over the MLP pair, 15 % of the tokens fire
        _stack("pair_batch4", "pair", 4096, 16384, 256, 4, 1),
        _stack("pair_batch64", "pair", 4096, 16384, 256, 64, 10),
        # a ragged batch of bf16 activations through a smaller block
        _stack("block_batch23_bf16x", "block", 2560, 10240, 128, 23, 3, x="bf16"),
        # prefill of a block, bf16 activations, a fifth of the tokens fires
        _stack("block_prefill2048", "block", 4096, 16384, 512, 2048, 410, x="bf16"),
        # a short ragged prompt, fp32 activations
        _stack("pair_prefill333", "pair", 4096, 16384, 256, 333, 50),
        # what a model pays once per block: six images and the four E of the single-pass gate
        {"name": "prepare_block", "kind": "prepare", "shape": "block", "d": 4096, "ffn": 16384, "k": 256, "w": "bf16"},
        # a sequence's first new direction: the basis of q, k, v and its images grow by one column (the column of
        # the sequence before is dropped first, as a serving loop does that starts from the calibrated basis)
        {"name": "extend_qkv", "kind": "extend", "d": 4096, "k": 256, "cap": 512, "m": 4096, "maps": 3, "w": "bf16"},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _mult(x, q):
    return max(q, int(x / q + 0.5) * q)


def draw(rng):
    kind = rng.choice(["f32", "token", "token", "layers", "batch", "batch", "prefill", "prefill", "prepare", "extend"])
    d = _mult(_log(rng, 1024, 5120), 128)
    ffn = _mult(d * rng.uniform(2.5, 4.0), 128)
    rank = rng.choice([64, 128, 256, 512])
    ragged_rank = rng.choice([rank, _mult(_log(rng, 48, 384), 8)])
    rank, ragged_rank = min(rank, d // 4), min(ragged_rank, d // 4)
    if kind == "f32":   # one fp32 map, any number of output rows, one token to a small batch
        d = _mult(_log(rng, 384, 2048), 64)
        tokens = int(_log(rng, 1, 64.99))
        return _stack("", "one", d, int(_log(rng, 700, 8192)), rng.choice([32, 64, 96, 128]) if d >= 512 else 64, tokens,
                      max(1, round(0.25 * tokens)), w="f32", call="separate")
    if kind == "token":  # one block or pair, explicit gate, either no input or one fires
        shape = rng.choice(["block", "pair"])
        return _stack("", shape, d, ffn, ragged_rank, 1, rng.choice([0, 0, 3 if shape == "block" else 2]),
                      x=rng.choice(["f32", "bf16"]))
    if kind == "layers":  # blocks of one call, single-pass gate
        return _stack("", "block", d, ffn, rng.choice([64, 128, 256]), 1, rng.choice([0, 21, 5]),
                      layers=int(_log(rng, 1, 16.99)), gate="single", slow=rng.choice(["mc_wr", "wx"]),
                      image=rng.choice(["same", "fp8"]), call=rng.choice(["run", "plan"]))
    if kind == "batch":  # decode batches
        tokens = int(_log(rng, 2, 128.99))
        return _stack("", rng.choice(["block", "pair"]), d, ffn, ragged_rank, tokens, round(0.15 * tokens),
                      x=rng.choice(["f32", "f32", "bf16"]))
    if kind == "prefill":
        tokens = int(_log(rng, 129, 2048.99))
        return _stack("", rng.choice(["block", "pair"]), min(d, 4096), min(ffn, 16384), rng.choice([64, 128, 192, 256, 384, 512])
                      if d >= 2048 else rank, tokens, round(rng.uniform(0.0, 0.3) * tokens), x=rng.choice(["f32", "bf16"]))
    if kind == "prepare":
        return {"kind": "prepare", "shape": "block", "d": min(d, 4096), "ffn": min(ffn, 16384), "k": rank, "w": "bf16"}
    k = rank // 2
    return {"kind": "extend", "d": d, "k": k, "cap": 2 * k, "m": rng.choice([d, ffn]), "maps": rng.randint(1, 3),
            "w": "bf16"}


# ------------------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _weight(m, d, dtype, gen):
    return torch.randn((m, d), generator=gen, device=DEV).mul_(1.0 / math.sqrt(d)).to(dtype)


def _basis(d, k, gen):
    """Orthonormal [d, k] in fp64: the polar factor of a Gaussian by Newton's iteration (k is at most d / 4, where the
    singular values start between 1/2 and 3/2)."""
    q = torch.randn((d, k), generator=gen, device=DEV, dtype=torch.float64) / math.sqrt(d)
    for _ in range(8):
        q = 1.5 * q - 0.5 * (q @ (q.T @ q))
    return q


def _tokens(U64, fired, gen, p=1.5):
    """X[T, d] fp64 with residual ratio EPS (1.2 .. 4.2) for fired tokens and EPS (0.2 .. 0.8) for the others."""
    d, k = U64.shape
    T = fired.shape[0]
    f64 = dict(generator=gen, device=DEV, dtype=torch.float64)
    lam = torch.arange(1, k + 1, device=DEV, dtype=torch.float64) ** (-p)
    a = torch.randn((T, k), **f64) * torch.sqrt(lam)[None, :]
    u = torch.rand(T, **f64)
    rho = torch.where(fired, EPS * (1.2 + 3.0 * u), EPS * (0.2 + 0.6 * u))
    n = torch.randn((T, d), **f64)
    for _ in range(2):
        n = n - (n @ U64) @ U64.T
    n = n / torch.linalg.norm(n, dim=1, keepdim=True)
    return a @ U64.T + (rho * torch.linalg.norm(a, dim=1) / torch.sqrt(1.0 - rho * rho))[:, None] * n


def _product(W, U):
    """W U in 64 bits, some rows of W at a time."""
    U64 = U.double()
    return torch.cat([W[i:i + 4096].double() @ U64 for i in range(0, W.shape[0], 4096)])


def _fp8(M):
    """E4M3 codes and power-of-two row scales of a stored image."""
    top = M.float().abs().amax(dim=1) / 448.0
    mant, ex = torch.frexp(top)
    ex = torch.where(mant == 0.5, ex - 1, ex)
    scale = torch.ldexp(torch.ones_like(top), ex)
    return (M.float() / scale[:, None]).to(torch.float8_e4m3fn).view(torch.uint8).contiguous(), scale


def _widths(case):
    for name, maps in SHAPES[case["shape"]]:
        yield case[name], [case[m] for m in maps]


def _inputs(case, seed):
    """Yields (U, X, [(W, M, codes, scale)]) for every input of a "stack" case, in the order of the call."""
    dt, B, salt = TORCH[case["w"]], case["tokens"], 0
    for _ in range(case["layers"]):
        for d, maps in _widths(case):
            gen = _gen(seed, salt)
            fired = torch.zeros(B, dtype=torch.bool, device=DEV)
            if B == 1:
                step = case["fired"]
                fired[0] = step > 0 and salt % step == min(5, step - 1)
            else:
                fired[torch.randperm(B, generator=gen, device=DEV)[:case["fired"]]] = True
            U64 = _basis(d, case["k"], gen)
            X = _tokens(U64, fired, gen).to(TORCH[case["x"]]).contiguous()
            U = U64.to(dt)
            out = []
            for m in maps:
                W = _weight(m, d, dt, gen)
                M = _product(W, U).to(dt)
                codes, scale = _fp8(M) if case["image"] == "fp8" else (None, None)
                out.append((W, M, codes, scale))
            salt += 1
            yield U, X, out


def _gram(U):
    return (U.double().T @ U.double() - torch.eye(U.shape[1], device=DEV, dtype=torch.float64))


def _carve(sizes, dtype):
    """One buffer and a view of it for each size."""
    flat = torch.zeros(sum(sizes), dtype=dtype, device=DEV)
    return flat, list(torch.split(flat, sizes))


def _prepare_stack(case, seed):
    inputs, maps = [], []
    flags = (gsi.INPUT_GATE_SINGLE_PASS if case["gate"] == "single" else 0) | \
            (gsi.INPUT_SLOW_PATH_WX if case["slow"] == "wx" else 0)
    for i, (U, X, ms) in enumerate(_inputs(case, seed)):
        inputs.append({"U": U, "X": X, "flags": flags,
                       "gram": _gram(U).float().contiguous() if case["gate"] == "single" else None})
        for W, M, codes, scale in ms:
            maps.append({"W": W, "M": M if codes is None else codes, "M_scale": scale, "input_id": i})
    names = ["C", "rnorm", "xnorm", "mask", "fired_idx", "n_fired"] + (["R"] if case["gate"] == "explicit" else [])
    if case["layers"] > 1:  # the results of a whole model lie in one buffer of each kind
        flat, views = _carve([mp["W"].shape[0] for mp in maps], torch.float32)
        for mp, y in zip(maps, views):
            mp["Y"] = y[None, :]
        st = gsi.LayerStack(inputs, maps, case["tokens"], EPS)
        out = [flat]
        for n in names:
            flat, views = _carve([t[n].numel() for t in st.inputs_t], st.inputs_t[0][n].dtype)
            for t, v in zip(st.inputs_t, views):
                t[n] = v.view(t[n].shape)
            out.append(flat)
        st.refresh()
    else:
        st = gsi.LayerStack(inputs, maps, case["tokens"], EPS)
        out = [t["Y"] for t in st.maps_t] + [t[n] for t in st.inputs_t for n in names]
    plan = st.build_plan() if case["call"] == "plan" else None
    return {"case": case, "stack": st, "plan": plan, "out": out}


def _maps(shape_case, seed):
    """(U, [W]) of every input of a "prepare" case."""
    for salt, (d, maps) in enumerate(_widths(shape_case)):
        gen = _gen(seed, salt)
        dt = TORCH[shape_case["w"]]
        yield _basis(d, shape_case["k"], gen).to(dt), [_weight(m, d, dt, gen) for m in maps]


def _extend_inputs(case, seed):
    gen = _gen(seed, 0)
    dt, d, k, cap = TORCH[case["w"]], case["d"], case["k"], case["cap"]
    U = torch.zeros((d, cap), device=DEV, dtype=dt)
    U64 = _basis(d, k, gen)
    U[:, :k] = U64.to(dt)
    x = _tokens(U64, torch.ones(1, dtype=torch.bool, device=DEV), gen)
    u = U.double()
    r = x - (x @ u) @ u.T
    maps = []
    for _ in range(case["maps"]):
        W = _weight(case["m"], d, dt, gen)
        maps.append((W, _product(W, U).to(dt)))
    norm = lambda v: torch.linalg.norm(v, dim=1).float()
    return U, r[0].float().contiguous(), norm(r), norm(x), maps


def prepare(case, seed):
    if case["kind"] == "stack":
        return _prepare_stack(case, seed)
    if case["kind"] == "prepare":
        layers = []
        for U, Ws in _maps(case, seed):
            k = U.shape[1]
            layers.append((U, Ws, [torch.empty((W.shape[0], k), dtype=W.dtype, device=DEV) for W in Ws],
                           torch.empty((k, k), device=DEV)))
        return {"case": case, "layers": layers}
    U, R, rnorm, xnorm, maps = _extend_inputs(case, seed)
    i32 = dict(dtype=torch.int32, device=DEV)
    ws = torch.empty(int(gsi.lib.gsi_extend_basis_workspace_bytes(case["d"], case["cap"])), dtype=torch.uint8, device=DEV)
    return {"case": case, "U": U, "R": R, "rnorm": rnorm, "xnorm": xnorm, "maps": maps, "gram": _gram(U).float(),
            "k_cur": torch.zeros(1, **i32), "extended": torch.zeros(1, **i32), "ws": ws}


# ------------------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["kind"] == "stack":
        st = state["stack"]
        if case["call"] == "plan":
            st.run_plan(state["plan"][0])
        elif case["call"] == "run":
            st.run()
        else:
            for i, t in enumerate(st.inputs_t):
                gsi.project(t["U"], t["X"], t["C"], t["R"], t["rnorm"], t["xnorm"])
                gsi.gate(t["rnorm"], t["xnorm"], EPS, t["mask"], t["fired_idx"], t["n_fired"])
                for mp in st.maps_t:
                    if mp["input_id"] == i:
                        gsi.gated_linear(mp["W"], mp["M"], t["C"], t["R"], t["fired_idx"], t["n_fired"], mp["Y"])
        return state["out"]
    if case["kind"] == "prepare":
        out = []
        for U, Ws, Ms, E in state["layers"]:
            for W, M in zip(Ws, Ms):
                gsi.build_image(W, U, M)
            gsi.build_gram(U, E)
            out += Ms + [E]
        return out
    s = state
    s["U"][:, case["k"]].zero_()
    s["k_cur"].fill_(case["k"])
    gsi.extend_basis(s["U"], s["k_cur"], s["R"], s["rnorm"], s["xnorm"], EPS, s["maps"], s["gram"], s["extended"], s["ws"])
    return [s["U"], s["k_cur"], s["extended"], s["gram"]] + [M for _, M in s["maps"]]


# ------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and what its results may differ by
# ------------------------------------------------------------------------------------------------------------
def work(case):
    e = SIZE[case["w"]]
    by = fl = 0
    if case["kind"] == "stack":
        B, k, i = case["tokens"], case["k"], 0
        xs, img = SIZE[case["x"]], 1 if case["image"] == "fp8" else e
        single, wx = case["gate"] == "single", case["slow"] == "wx"
        for _ in range(case["layers"]):
            for d, maps in _widths(case):
                step = case["fired"]
                nf = step if B > 1 else int(step > 0 and i % step == min(5, step - 1))
                i += 1
                by += d * k * e + B * (d * xs + 4 * k) + (4 * k * k if single else 0)
                by += 0 if single and not nf else 4 * B * d
                fl += 2 * d * k * B * (1 if single else 2)
                for m in maps:
                    skip = single and wx and nf
                    by += (0 if skip else m * k * img) + (m * d * e if nf else 0) + 4 * B * m
                    fl += 2 * m * k * B + 2 * m * d * nf
    elif case["kind"] == "prepare":
        k = case["k"]
        for d, maps in _widths(case):
            by += d * k * e + 4 * k * k
            fl += 2 * d * k * k
            for m in maps:
                by += m * d * e + m * k * e
                fl += 2 * m * d * k
    else:
        d, k, m, n = case["d"], case["k"], case["m"], case["maps"]
        by = d * k * e + 4 * d + n * (m * d * e + m * e) + d * e + 8 * k
        fl = 6 * d * k + 2 * n * m * d
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """About four times what the path shows against exact()."""
    if case["kind"] == "prepare":   # images are rounded to bf16 once (1.7e-3 against the unrounded product)
        return {"rel": 4e-3}
    if case["kind"] == "extend":    # one rounded column among many (1.0e-4 .. 1.5e-4 of the whole array)
        return {"rel": 6e-4}
    # 32-bit sums; the largest figure is the residual's, whose terms cancel to a few percent (7e-5).  In batches of
    # more than 128 tokens r enters its product rounded to bf16 (1.3e-4 of y)
    return {"rel": 6e-4 if case["tokens"] > 128 else 3e-4}


# ------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------------------------
def _apply(W, v):
    """v W^T in 64 bits, some rows of W at a time."""
    return torch.cat([v @ W[i:i + 4096].double().T for i in range(0, W.shape[0], 4096)], dim=1)


def exact(case, seed):
    if case["kind"] == "prepare":
        out = []
        for U, Ws in _maps(case, seed):
            out += [_product(W, U) for W in Ws] + [_gram(U)]
        return out
    if case["kind"] == "extend":
        U, R, rnorm, xnorm, maps = _extend_inputs(case, seed)
        k, u = case["k"], U.double()
        r = R.double()
        r = r - u @ (u.T @ r)
        v = (r / torch.linalg.norm(r)).to(U.dtype)   # the images and E are those of the stored column
        U2, E = u.clone(), _gram(U)
        U2[:, k] = r / torch.linalg.norm(r)
        U[:, k] = v
        col = U.double().T @ v.double()
        col[k] -= 1.0
        E[k, :] = col
        E[:, k] = col
        out = [U2, torch.tensor([k + 1]), torch.tensor([1]), E]
        for W, M in maps:
            M2 = M.double()
            M2[:, k] = _apply(W, v.double()[None, :])[0]
            out.append(M2)
        return out
    ys, ins = [], []  # ins: one list of values per input
    for U, X, ms in _inputs(case, seed):
        u, x = U.double(), X.double()
        C = x @ u
        R = x - C @ u.T
        rn, xn = torch.linalg.norm(R, dim=1), torch.linalg.norm(x, dim=1)
        mask = rn >= EPS * xn
        idx = torch.nonzero(mask)[:, 0]
        fired_idx = torch.zeros(case["tokens"], dtype=torch.int32, device=DEV)
        fired_idx[:idx.numel()] = idx.to(torch.int32)
        for W, M, codes, scale in ms:
            m64 = M.double() if codes is None else codes.view(torch.float8_e4m3fn).double() * scale.double()[:, None]
            Y = C @ m64.T
            if idx.numel():
                add = _apply(W, x[idx] if case["slow"] == "wx" else R[idx])
                Y[idx] = add if case["slow"] == "wx" else Y[idx] + add
            ys.append(Y)
        ins.append([C, rn, xn, mask.to(torch.uint8), fired_idx, torch.tensor([idx.numel()], device=DEV)] +
                   ([R] if case["gate"] == "explicit" else []))
    if case["layers"] > 1:
        return [torch.cat([v.flatten() for v in part]) for part in [ys] + [list(p) for p in zip(*ins)]]
    return ys + [v for part in ins for v in part]
