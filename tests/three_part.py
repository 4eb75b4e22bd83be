"""Float64 emulation of the float32 layer with one planted mistake in the three-part
products, for tests of what the float32 kernels keep.

Float32 operands enter the matrix cores as three bfloat16 parts p0 + p1 + p2 and a product
takes the part products (i, j) with i + j <= 2.  `run` computes the layer's forward and
backward in float64; `plant` = (contraction, kind) drops in one contraction the third part
of its first operand ("a") or of its second ("b"), or the product of the second parts
("p11").  Each such mistake costs about 2^-18 of what it touches, as little as the rounding
of a float32 run of the same sums, so no bar on the size of an error tells the two apart.
Its pattern does: `share` is the coefficient of that pattern in an error, about one with
the mistake and about zero without, whatever the size of the (unrelated) rounding.
"""
import numpy as np

from oracle.backward import token_backward
from oracle.physics_attention import token_attention

FORWARD = ("P1.logits", "P1.sum", "P2.logits", "P2.decode")
BACKWARD = ("G.logits", "G.sum", "DX.logits", "DX.gZ", "DX.x_ds", "DX.dz_W2", "DX.w_ds", "DW2.sum")
KINDS = ("a", "b", "p11")


def bf16(v):
    u = np.asarray(v, np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32).astype(np.float64)


def two_parts(v):
    v = np.asarray(v, np.float32).astype(np.float64)
    p0 = bf16(v)
    return p0, bf16(v - p0)


def _product(a, b, contract, kind):
    if kind == "a":
        return contract(sum(two_parts(a)), b)
    if kind == "b":
        return contract(a, sum(two_parts(b)))
    if kind == "p11":
        return contract(a, b) - contract(two_parts(a)[1], two_parts(b)[1])
    return contract(a, b)


def run(x, g, W, H, M, inv_tau, plant=None, backward=True, stored_bf16=False):
    """Outputs of the layer as a dict; with stored_bf16 the slice logits' weights are rounded to
    bfloat16, as bf16 storage keeps them."""
    kind = dict([plant]) if plant else {}
    N, C = x.shape
    dh = C // H
    W = {k: np.asarray(v, np.float64) for k, v in W.items()}
    scale = np.log2(np.e) * inv_tau
    W2s, b2s = W["W2"] * scale, W["b2"] * scale
    if stored_bf16:
        W2s = bf16(W2s)

    def weights(name):
        L = (_product(x, W2s, lambda a, b: a @ b, kind.get(name)) + b2s).reshape(N, H, M)
        e = np.exp2(L - L.max(axis=2, keepdims=True))
        return e / e.sum(axis=2, keepdims=True)

    def points_to_slices(w, v, k):  # sum over points
        return _product(w, v, lambda a, b: np.einsum("nhm,nc->hmc", a, b, optimize=True), k)

    def slices_to_points(w, v, k):  # sum over heads and slices
        return _product(w, v, lambda a, b: np.einsum("nhm,hmc->nc", a, b, optimize=True), k)

    def rows_dot(p, v, k):          # sum over channels
        return _product(p, v, lambda a, b: np.einsum("nc,hmc->nhm", a, b, optimize=True), k)

    w = weights("P1.logits")
    k = kind.get("P1.sum")
    s_raw = points_to_slices(w, x, k)
    d = (sum(two_parts(w)) if k == "a" else w).sum(axis=0)  # the same parts times one
    mean = s_raw / d[:, :, None]
    s = np.stack([mean[h] @ W["W1"][:, h * dh:(h + 1) * dh] + W["b1"][h * dh:(h + 1) * dh] for h in range(H)])
    s1 = token_attention(s, W["Wq"], W["Wk"], W["Wv"])
    Z = np.stack([s1[h] @ W["W3"][h * dh:(h + 1) * dh] for h in range(H)])
    out = {"s_raw": s_raw, "d": d,
           "out": slices_to_points(weights("P2.logits"), Z + W["b3"] / H, kind.get("P2.decode"))}
    if not backward:
        return out
    dZ = points_to_slices(weights("G.logits"), g, kind.get("G.sum"))
    ds_raw, dd, grads = token_backward({"s_raw": s_raw, "d": d, "s": s, "s1": s1}, dZ, W, H)
    out.update(grads, db3=dZ[0].sum(axis=0))
    w = weights("DX.logits")
    dw = rows_dot(g, Z, kind.get("DX.gZ")) + rows_dot(x, ds_raw, kind.get("DX.x_ds")) + dd[None]
    dz = inv_tau * w * (dw - (w * dw).sum(axis=2, keepdims=True))
    dz2 = dz.reshape(N, H * M)
    out["dx"] = (_product(dz2, W["W2"], lambda a, b: a @ b.T, kind.get("DX.dz_W2"))
                 + slices_to_points(w, ds_raw, kind.get("DX.w_ds")))
    k = kind.get("DW2.sum")
    out["dW2"] = _product(dz2, x, lambda a, b: b.T @ a, k)
    out["db2"] = (sum(two_parts(dz2)) if k == "a" else dz2).sum(axis=0)
    return out


def case(C, H, M, N, bf16_storage=False):
    """(x, g, W) of a case: slice logits four times as wide as Xavier's, so that the slices differ
    enough for every contraction to reach an output."""
    from ts3_synth import make_weights
    rng = np.random.default_rng(N)
    x, g = (rng.standard_normal((N, C)).astype(np.float32).astype(np.float64) for _ in range(2))
    W = make_weights(C, H, M, C // H, seed=2, bias_seed=3)
    W["W2"] = W["W2"] * np.float32(4)
    return (bf16(x) if bf16_storage else x), g, W


def pattern(ref, planted, outputs):
    """(name, pattern) of the output in which a planted mistake stands out most: the one with the
    largest relative size times the root of its number of values (which is how well a sum over the
    values separates it from rounding of a given relative size)."""
    def weight(k):
        e = planted[k] - ref[k]
        return np.linalg.norm(e) / np.linalg.norm(ref[k]) * np.sqrt(e.size)
    name = max(outputs, key=weight)
    return name, planted[name] - ref[name]


def share(error, pat):
    return float((error * pat).sum() / (pat * pat).sum())
