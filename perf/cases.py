"""Work that a user of the library has it do, as measurable cases.

Each case is one call (or one short sequence of calls) through the public Python
classes: ``PhysicsAttention`` (the layer), ``TransolverStack`` (the block stack).
``listed()`` gives fixed cases, ``draw()`` more of the same ranges; ``prepare()``
makes what a program holds before the call, ``run()`` makes the call, and
``exact()`` gives the same outputs in float64 from plain torch.

Kinds of case:
  layer   one Physics-Attention layer over a resident mesh (forward)
  stream  the same layer with the mesh arriving tile by tile (accumulate, finalize,
          attention), then decoded chunk by chunk
  decode  query points decoded from a state that the program keeps
  train   forward and backward of the layer in float32
  stack   the pre-norm block stack over a mesh (one whole model call)
  query   query points through every block of a stack from its cached states
  ffn     the feed-forward half of one block

Points are uniform in a box; their features are the Fourier features of the
coordinates under a Gaussian map, normalised per point, as the model's input
embedding gives them.  Weights are Xavier-uniform with small random biases, the slice
logits' map twice as wide so that the slices differ as they do after training.
"""
import math

import torch

TAU = 0.5


def listed():
    return [
        # the smallest mesh of the library's workloads: a 4,096-point surface in one
        # tile and one span, float32; launches and latency decide
        dict(name="layer_4k_fp32", kind="layer", C=64, H=4, M=16, dtype="fp32", N=4096, Q=4096, tile=4096,
             chunk=4096, accum="fp32"),
        # a surface mesh of ordinary size (ragged) with the default span length
        dict(name="layer_100k_bf16", kind="layer", C=128, H=8, M=64, dtype="bf16", N=100_003, Q=32_768,
             tile=1_015_808, chunk=1_000_000, accum="fp32"),
        # the volume mesh of the benchmark, one layer at its tile, chunk and span sizes
        dict(name="layer_16m_bf16", kind="layer", C=128, H=8, M=64, dtype="bf16", N=16_000_000, Q=15_625,
             tile=1_000_000, chunk=1_000_000, accum="fp32"),
        # a float32 forward at the 8-block model's width (no half-precision storage)
        dict(name="layer_c256_fp32", kind="layer", C=256, H=8, M=64, dtype="fp32", N=30_000, Q=4096,
             tile=32_768, chunk=30_000, accum="fp32"),
        # a layer of a width that is no power of two, bf16, ragged
        dict(name="layer_c192_bf16", kind="layer", C=192, H=4, M=48, dtype="bf16", N=50_021, Q=4096,
             tile=16_384, chunk=20_000, accum="fp32"),
        # a 1M-point surface that arrives in 65,536-point tiles, sums folded in float64
        dict(name="stream_1m_bf16", kind="stream", C=128, H=8, M=32, dtype="bf16", N=1_000_000, Q=16_384,
             tile=65_536, chunk=65_536, accum="fp64"),
        # a serving request: a few thousand query points against a kept state
        dict(name="decode_5k_bf16", kind="decode", C=128, H=8, M=64, dtype="bf16", N=5003, Q=4096, mesh=65_536,
             accum="fp32"),
        # a training step on a small, ragged subset
        dict(name="train_60k_fp32", kind="train", C=128, H=8, M=64, dtype="fp32", N=60_001, Q=15_625,
             tile=1_000_000, chunk=1_000_000, accum="fp32"),
        # the training step of the benchmark: a 2M-point subset
        dict(name="train_2m_fp32", kind="train", C=128, H=8, M=64, dtype="fp32", N=2_000_000, Q=15_625,
             tile=1_000_000, chunk=1_000_000, accum="fp32"),
        # the 8-block model over a surface mesh
        dict(name="stack_1m_bf16", kind="stack", C=256, H=8, M=64, L=8, F=1024, N=1_000_000, Q=31_250,
             tile=1_000_000, chunk=1_000_000, accum="fp32"),
        # a serving request to the whole model: query points from the cached states
        dict(name="query_4k_bf16", kind="query", C=256, H=8, M=64, L=8, F=1024, N=4096, Q=4096, mesh=32_768,
             chunk=4096, accum="fp32"),
        # one block's feed-forward half at the narrower model's width, ragged
        dict(name="ffn_250k_bf16", kind="ffn", C=128, H=8, M=32, F=512, N=250_001, Q=16_384, accum="fp32"),
    ]


BF16_SHAPES = [(64, 4, 16), (64, 4, 32), (128, 8, 16), (128, 8, 32), (128, 8, 64), (128, 2, 64), (256, 8, 64)]
FP32_SHAPES = [(64, 4, 16), (64, 4, 32), (128, 8, 16), (128, 8, 32), (128, 8, 64)]
# shapes outside the tuned lists (multiples of 16)
ODD_SHAPES = [(192, 4, 48, "bf16"), (192, 4, 48, "fp32"), (96, 6, 16, "fp32"), (48, 1, 80, "fp32"),
              (256, 8, 64, "fp32"), (128, 8, 128, "bf16"), (512, 8, 16, "bf16")]
STACK_SHAPES = [(128, 8, 32, 512), (128, 8, 64, 512), (256, 8, 64, 1024)]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["layer", "layer", "layer", "odd", "stream", "decode", "train", "stack", "query", "ffn"])
    Q = rng.choice([1024, 4096, 15_625, 16_384, 32_768])
    accum = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "odd":
        C, H, M, dtype = rng.choice(ODD_SHAPES)
        n = size(500, 50_000)
        return dict(kind="layer", C=C, H=H, M=M, dtype=dtype, N=n, Q=rng.choice([1024, 4096]), tile=16_384,
                    chunk=rng.choice([10_000, 65_536]), accum=accum)
    if kind in ("layer", "stream", "decode"):
        dtype = rng.choice(["bf16", "bf16", "fp32"])
        C, H, M = rng.choice(BF16_SHAPES if dtype == "bf16" else FP32_SHAPES)
        if kind == "decode":
            return dict(kind=kind, C=C, H=H, M=M, dtype=dtype, N=size(1, 300_000), Q=4096, mesh=size(1000, 65_536),
                        accum=accum)
        n = size(1000, 4_000_000 if dtype == "bf16" else 1_000_000)
        return dict(kind=kind, C=C, H=H, M=M, dtype=dtype, N=n, Q=Q, tile=Q * max(1, rng.choice([65_536, 1_000_000]) // Q),
                    chunk=rng.choice([65_536, 1_000_000]), accum=accum)
    if kind == "train":
        C, H, M = rng.choice(FP32_SHAPES)
        return dict(kind=kind, C=C, H=H, M=M, dtype="fp32", N=size(2000, 1_000_000), Q=Q,
                    tile=Q * max(1, rng.choice([65_536, 1_000_000]) // Q), chunk=1_000_000, accum=accum)
    C, H, M, F = rng.choice(STACK_SHAPES)
    if kind == "stack":
        return dict(kind=kind, C=C, H=H, M=M, L=rng.randint(2, 8), F=F, N=size(2000, 500_000), Q=Q,
                    tile=Q * max(1, rng.choice([65_536, 1_000_000]) // Q), chunk=rng.choice([65_536, 1_000_000]),
                    accum=accum)
    if kind == "query":
        return dict(kind=kind, C=C, H=H, M=M, L=rng.randint(2, 8), F=F, N=size(1, 30_000), Q=4096, mesh=32_768,
                    chunk=32_768, accum=accum)
    return dict(kind="ffn", C=C, H=H, M=M, F=F, N=size(500, 1_000_000), Q=16_384, accum=accum)


# ------------------------------------------------------------------ inputs

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 64 + stream)
    return g


def _features(n, C, dtype, seed, stream=0):
    """Rows of the model's input embedding for n points, [n, C]."""
    g = _gen(seed, stream)
    R = torch.randn((96, C), generator=_gen(seed, 63), device="cuda") / math.sqrt(96.0)
    f = math.pi * 2.0 ** (torch.arange(16, device="cuda") / 3.0)
    x = torch.empty((n, C), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    for a in range(0, n, 1 << 20):
        b = min(n, a + (1 << 20))
        q = torch.rand((b - a, 3), generator=g, device="cuda") * 2.0 - 1.0
        arg = q[:, :, None] * f
        z = torch.cat([arg.sin(), arg.cos()], dim=2).reshape(b - a, 96) @ R
        x[a:b] = torch.nn.functional.layer_norm(z, (C,)).to(x.dtype)
    return x


def _weights(case, seed, block=0):
    """Float32 weights of one layer (and, for the stack kinds, of one block)."""
    C, H, M = case["C"], case["H"], case["M"]
    dh, HM = C // H, H * M
    g = _gen(seed, 8 + block)

    def uniform(shape, bound):
        return (torch.rand(shape, generator=g, device="cuda") * 2.0 - 1.0) * bound

    def xavier(*shape):
        return uniform(shape, math.sqrt(6.0 / (shape[-2] + shape[-1])))

    w = dict(W2=2.0 * xavier(C, HM), W1=xavier(C, C), Wq=xavier(H, dh, dh), Wk=xavier(H, dh, dh), Wv=xavier(H, dh, dh),
             W3=xavier(C, C), b2=uniform((HM,), 0.1), b1=uniform((C,), 0.1), b3=uniform((C,), 0.1))
    if "F" in case:
        F = case["F"]
        w.update(Wa=xavier(C, F), Wb=xavier(F, C), ba=uniform((F,), 0.1), bb=uniform((C,), 0.1))
        for ln in ("ln1", "ln2"):
            w[ln + "_g"] = 1.0 + uniform((C,), 0.1)
            w[ln + "_b"] = uniform((C,), 0.1)
    return w


def prepare(case, seed):
    from paper_2602_04940_amd import LayerWeights, PhysicsAttention
    from paper_2602_04940_amd.stack import BlockWeights, TransolverStack
    kind, C, H, M, N = case["kind"], case["C"], case["H"], case["M"], case["N"]
    s = {"case": case}
    if kind in ("stack", "query", "ffn"):
        blocks = 2 if kind == "ffn" else case["L"]
        s["x"] = _features(N, C, "bf16", seed)
        s["blocks"] = [BlockWeights(_weights(case, seed, l)) for l in range(blocks)]
        points = max(N, case.get("mesh", 0))
        s["model"] = TransolverStack(C, H, M, blocks, hidden=case["F"], temperature=TAU, group_span=case["Q"],
                                     max_points=points, accum=case["accum"])
        if kind == "query":
            mesh = _features(case["mesh"], C, "bf16", seed, 1)
            s["model"].forward(s["blocks"], mesh, tile=case["Q"] * max(1, case["mesh"] // case["Q"]), chunk=case["mesh"])
        if kind == "ffn":
            s["pa"] = _features(N, C, "bf16", seed, 1)
            s["next"] = torch.empty_like(s["x"])
        return s
    s["w"] = LayerWeights(_weights(case, seed))
    s["x"] = _features(N, C, case["dtype"], seed)
    s["out"] = torch.empty_like(s["x"])
    s["layer"] = PhysicsAttention(C, H, M, temperature=TAU, dtype=case["dtype"], group_span=case["Q"],
                                  max_points=max(N, case.get("mesh", 0)), accum=case["accum"])
    if kind == "decode":
        mesh = _features(case["mesh"], C, case["dtype"], seed, 1)
        s["layer"].forward(s["w"], mesh, tile=case["Q"] * max(1, case["mesh"] // case["Q"]))
    if kind == "train":
        s["g"] = torch.randn((N, C), generator=_gen(seed, 2), device="cuda")
    return s


# ------------------------------------------------------------------ the call

def run(state):
    case, x = state["case"], state["x"]
    kind = case["kind"]
    if kind == "layer":
        return state["layer"].forward(state["w"], x, tile=case["tile"], chunk=case["chunk"], out=state["out"])
    if kind == "stream":
        layer, w, out = state["layer"], state["w"], state["out"]
        n, tile, chunk = x.shape[0], case["tile"], case["chunk"]
        layer.reset()
        for a in range(0, n, tile):
            layer.accumulate(w, x[a:a + tile], a)
        layer.finalize(w)
        layer.attention(w)
        for a in range(0, n, chunk):
            layer.deslice(w, x[a:a + chunk], out[a:a + chunk])
        return out
    if kind == "decode":
        return state["layer"].deslice(state["w"], x, state["out"])
    if kind == "train":
        layer, w = state["layer"], state["w"]
        out = layer.forward(w, x, tile=case["tile"], chunk=case["chunk"], out=state["out"])
        dx, grads = layer.backward(w, x, state["g"], tile=case["tile"])
        return {"out": out, "dx": dx, **grads}
    y = x.clone()  # the stack works in place; the program keeps its features
    if kind == "stack":
        return state["model"].forward(state["blocks"], y, tile=case["tile"], chunk=case["chunk"])
    if kind == "query":
        return state["model"].decode(state["blocks"], y, chunk=case["chunk"])
    return {"x": state["model"].feedforward(state["blocks"], 0, y, state["pa"], state["next"]), "next": state["next"]}


# ------------------------------------------------------------------ what it takes

def work(case):
    """Bytes: inputs once, outputs once, weights once.  Flops: the logits once, and each
    contraction in the order of the linear maps that takes fewer products."""
    C, H, M, N = case["C"], case["H"], case["M"], case["N"]
    HM = H * M
    e = 4 if case.get("dtype") == "fp32" else 2
    logits, contract = 2.0 * C * HM, 2.0 * min(HM * C, C * C + M * C)
    layer = logits + 2 * contract
    wbytes = 4.0 * (C * HM + 2 * C * C + 3 * C * (C // H) + HM + 2 * C)
    ffn = 4.0 * C * case.get("F", 0)
    wffn = 8.0 * C * case.get("F", 0)
    kind = case["kind"]
    if kind == "decode":
        return {"bytes": 2.0 * N * C * e + 4.0 * (C * HM + HM * C), "flops": N * (logits + contract)}
    if kind == "train":
        # the forward's contractions, and six more with the slices of all heads
        return {"bytes": 4.0 * N * C * e + 3 * wbytes, "flops": N * (layer + 12.0 * C * HM)}
    if kind == "stack":
        return {"bytes": 2.0 * N * C * e + case["L"] * (wbytes + wffn), "flops": case["L"] * N * (layer + ffn)}
    if kind == "query":
        return {"bytes": 2.0 * N * C * e + case["L"] * (wbytes + wffn), "flops": case["L"] * N * (logits + contract + ffn)}
    if kind == "ffn":
        return {"bytes": 4.0 * N * C * e + wffn, "flops": N * ffn}
    return {"bytes": 2.0 * N * C * e + wbytes, "flops": N * layer}


def tolerance(case):
    """About four times what the path shows against float64 over these ranges."""
    kind = case["kind"]
    if kind == "train":
        return {"rel": 2e-5}
    if case.get("dtype") == "fp32":
        return {"rel": 5e-6}
    if kind in ("stack", "query"):
        return {"rel": 2e-2}
    return {"rel": 1.2e-2}


# ------------------------------------------------------------------ float64

STEP = 1 << 17


def _steps(n):
    return [(a, min(n, a + STEP)) for a in range(0, n, STEP)]


def _softmax(x, w, H, M):
    z = (x @ w["W2"] + w["b2"]).reshape(-1, H, M) / TAU
    return torch.softmax(z, dim=2).reshape(-1, H * M)


def _state(x, w, H, M):
    """Slice sums, slice tokens, attended tokens and decoding rows of the mesh x."""
    C = x.shape[1]
    dh = C // H
    s_raw = torch.zeros((H * M, C), device="cuda", dtype=torch.float64)
    d = torch.zeros((H * M,), device="cuda", dtype=torch.float64)
    for a, b in _steps(x.shape[0]):
        xa = x[a:b].double()
        p = _softmax(xa, w, H, M)
        s_raw += p.T @ xa
        d += p.sum(0)
    mean = s_raw / d[:, None]
    s, s1, Z, A = [], [], [], []
    for h in range(H):
        c, r = slice(h * dh, (h + 1) * dh), slice(h * M, (h + 1) * M)
        s.append(mean[r] @ w["W1"][:, c] + w["b1"][c])
        q, k, v = s[h] @ w["Wq"][h], s[h] @ w["Wk"][h], s[h] @ w["Wv"][h]
        A.append(torch.softmax(q @ k.T / math.sqrt(dh), dim=1))
        s1.append(A[h] @ v)
        Z.append(s1[h] @ w["W3"][c])
    return dict(d=d, mean=mean, s=s, s1=s1, A=A, Z=torch.cat(Z))


def _decode(x, w, Z, H, M):
    out = torch.empty(x.shape, device="cuda", dtype=torch.float64)
    for a, b in _steps(x.shape[0]):
        out[a:b] = _softmax(x[a:b].double(), w, H, M) @ Z + w["b3"]
    return out


def _ln(x, w, name):
    return torch.nn.functional.layer_norm(x, (x.shape[1],), w[name + "_g"], w[name + "_b"], 1e-5)


def _ffn(y, w):
    out = torch.empty_like(y)
    for a, b in _steps(y.shape[0]):
        h = torch.nn.functional.gelu(_ln(y[a:b], w, "ln2") @ w["Wa"] + w["ba"])
        out[a:b] = y[a:b] + h @ w["Wb"] + w["bb"]
    return out


def _blocks(x, blocks, H, M, Zs=None):
    """The stack over x; with Zs, decoded from those states.  Returns the output and the states."""
    made = []
    for l, w in enumerate(blocks):
        xn = _ln(x, w, "ln1")
        Z = _state(xn, w, H, M)["Z"] if Zs is None else Zs[l]
        made.append(Z)
        x = _ffn(x + _decode(xn, w, Z, H, M), w)
    return x, made


def _backward(x, g, w, H, M):
    C = x.shape[1]
    dh = C // H
    st = _state(x, w, H, M)
    f64 = dict(device="cuda", dtype=torch.float64)
    dZ = torch.zeros((H * M, C), **f64)
    for a, b in _steps(x.shape[0]):
        dZ += _softmax(x[a:b].double(), w, H, M).T @ g[a:b].double()
    r = {"db3": g.double().sum(0), "dW1": torch.zeros((C, C), **f64), "dW3": torch.zeros((C, C), **f64),
         "db1": torch.zeros((C,), **f64)}
    for n in ("dWq", "dWk", "dWv"):
        r[n] = torch.zeros((H, dh, dh), **f64)
    ds_raw = torch.zeros((H * M, C), **f64)
    dd = torch.zeros((H * M,), **f64)
    for h in range(H):
        c, rows = slice(h * dh, (h + 1) * dh), slice(h * M, (h + 1) * M)
        s, A, scale = st["s"][h], st["A"][h], 1.0 / math.sqrt(dh)
        q, k, v = s @ w["Wq"][h], s @ w["Wk"][h], s @ w["Wv"][h]
        ds1 = dZ[rows] @ w["W3"][c].T
        r["dW3"][c] = st["s1"][h].T @ dZ[rows]
        dA = ds1 @ v.T
        da = A * (dA - (dA * A).sum(1, keepdim=True)) * scale
        dq, dk, dv = da @ k, da.T @ q, A.T @ ds1
        r["dWq"][h], r["dWk"][h], r["dWv"][h] = s.T @ dq, s.T @ dk, s.T @ dv
        ds = dq @ w["Wq"][h].T + dk @ w["Wk"][h].T + dv @ w["Wv"][h].T
        r["dW1"][:, c] = st["mean"][rows].T @ ds
        r["db1"][c] = ds.sum(0)
        dmean = ds @ w["W1"][:, c].T
        ds_raw[rows] = dmean / st["d"][rows, None]
        dd[rows] = -(dmean * st["mean"][rows]).sum(1) / st["d"][rows]
    r["dx"] = torch.empty(x.shape, **f64)
    r["out"] = torch.empty(x.shape, **f64)
    r["dW2"] = torch.zeros((C, H * M), **f64)
    r["db2"] = torch.zeros((H * M,), **f64)
    for a, b in _steps(x.shape[0]):
        xa, ga = x[a:b].double(), g[a:b].double()
        p = _softmax(xa, w, H, M)
        dw = ga @ st["Z"].T + xa @ ds_raw.T + dd
        mean = (p * dw).reshape(-1, H, M).sum(2)
        dz = p * (dw - mean.repeat_interleave(M, dim=1)) / TAU
        r["dx"][a:b] = dz @ w["W2"].T + p @ ds_raw
        r["dW2"] += xa.T @ dz
        r["db2"] += dz.sum(0)
        r["out"][a:b] = p @ st["Z"] + w["b3"]
    return r


def exact(case, seed):
    kind, C, H, M, N = case["kind"], case["C"], case["H"], case["M"], case["N"]

    def weights(block=0):
        return {k: v.double() for k, v in _weights(case, seed, block).items()}

    x = _features(N, C, case.get("dtype", "bf16"), seed)
    if kind in ("layer", "stream"):
        w = weights()
        return _decode(x, w, _state(x, w, H, M)["Z"], H, M)
    if kind == "decode":
        w = weights()
        return _decode(x, w, _state(_features(case["mesh"], C, case["dtype"], seed, 1), w, H, M)["Z"], H, M)
    if kind == "train":
        g = torch.randn((N, C), generator=_gen(seed, 2), device="cuda")
        return _backward(x, g, weights(), H, M)
    if kind == "ffn":
        y = _ffn(x.double() + _features(N, C, "bf16", seed, 1).double(), weights(0))
        return {"x": y, "next": _ln(y, weights(1), "ln1")}
    blocks = [weights(l) for l in range(case["L"])]
    if kind == "stack":
        return _blocks(x.double(), blocks, H, M)[0]
    _, Zs = _blocks(_features(case["mesh"], C, "bf16", seed, 1).double(), blocks, H, M)
    return _blocks(x.double(), blocks, H, M, Zs)[0]
