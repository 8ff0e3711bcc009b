"""Timed cases of the library: the calls a program makes, over the range of sizes it makes them at.

A case is a dict of plain values.  ``kind`` names the public call:

  forward    Context.forward: pack, attention and unpack of every head chunk ([S][H][d] in and out)
  slots      Context.forward_slots: the same on two chunk slots
  attention  hcms.attention on head-major tensors
  train      HcmsAttention: a forward and its gradients through autograd
  linear     hcms.linear, a projection
  qkv        hcms.qkv_projection with the rotary embedding on a latent grid
  layer      Context.layer_forward: projection, chunk loop, output projection

S tokens, H local heads of dimension d, P sequence shards, D the model width; ``chunks`` is the
head chunking as text ("2,2,1"), ``grid`` the latent grid ("36,30,52", frames x rows x columns).
Queries, keys and values are standard normal (what a normalised projection gives), weights standard
normal over the square root of their input width, output gradients standard normal.
"""
import math

import torch

import paper_2607_01817_amd as hcms

DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}
BASE = 10000.0   # base of the rotary embedding's frequencies


def listed():
    return [
        # The smallest call: 512 tokens, 4 heads of 64, fp32 storage, two chunks.  Launches and
        # host time count.
        dict(name="forward_tiny_fp32", kind="forward", S=512, H=4, d=64, P=4, dtype="fp32",
             chunks="2,2"),
        # A short sequence, 4096 tokens and 8 heads in two chunks: fewer tiles than compute units.
        dict(name="forward_small", kind="forward", S=4096, H=8, d=128, P=8, dtype="bf16",
             chunks="4,4"),
        # The flagship: the 36-frame video share of one of 8 ranks, uneven chunks.
        dict(name="forward_wan_p8", kind="forward", S=56160, H=5, d=128, P=8, dtype="bf16",
             chunks="2,2,1"),
        # A 5-frame clip, one of 4 ranks, in the two-slot form used where memory is short.
        dict(name="slots_clip_p4", kind="slots", S=7800, H=10, d=128, P=4, dtype="bf16",
             chunks="5,5"),
        # A still image: one latent frame of 1560 tokens (no multiple of any tile), all 40 heads.
        dict(name="attention_image", kind="attention", S=1560, H=40, d=128, dtype="bf16",
             chunks="40"),
        # Heads of 64 at an ordinary length.
        dict(name="attention_d64", kind="attention", S=8192, H=16, d=64, dtype="bf16",
             chunks="8,8"),
        # A training step at an odd length without a score-gradient workspace.
        dict(name="train_ragged", kind="train", S=3001, H=8, d=128, P=1, dtype="bf16",
             chunks="4,4", ds_heads=0),
        # The flagship's training step, with the workspace for two heads per stream.
        dict(name="train_wan_p8", kind="train", S=56160, H=5, d=128, P=8, dtype="bf16",
             chunks="2,2,1", ds_heads=2),
        # The flagship's QKV projection with the rotation: a long reduction.
        dict(name="qkv_wan_p8", kind="qkv", grid="36,30,52", H=5, d=128, D=5120, dtype="bf16"),
        # One frame through a full-width projection: few row tiles, a long reduction.
        dict(name="linear_image", kind="linear", M=1560, N=5120, K=5120, dtype="bf16"),
        # A small whole layer: 240 tokens, five launches one after the other.
        dict(name="layer_small", kind="layer", grid="4,6,10", H=4, d=64, D=256, P=4, dtype="bf16",
             chunks="2,2"),
        # The flagship's whole layer.
        dict(name="layer_wan_p8", kind="layer", grid="36,30,52", H=5, d=128, D=5120, P=8,
             dtype="bf16", chunks="2,2,1"),
    ]


# ---------------------------------------------------------------------------
# Sizes
# ---------------------------------------------------------------------------
def _ints(text):
    return [int(x) for x in text.split(",")]


def _pairs(d, n):
    """The d / 2 pairs of a head vector in n groups, larger groups first (22, 21, 21 for 128)."""
    return [d // 2 // n + (1 if a < d // 2 % n else 0) for a in range(n)]


def _tokens(case):
    return math.prod(_ints(case["grid"])) if "grid" in case else case["S"]


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    k = case["kind"]
    if k == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": e * (M * K + N * K + M * N), "flops": 2 * M * N * K}
    S, H, d = _tokens(case), case["H"], case["d"]
    tensor, attn = e * S * H * d, 4 * S * S * H * d
    if k == "train":   # q, k, v and the output's gradient in; output and three gradients out
        return {"bytes": 8 * tensor, "flops": attn + 10 * S * S * H * d}
    if k in ("qkv", "layer"):
        D = case["D"]
        proj, w = 2 * S * D * 3 * H * d, e * 3 * H * d * D
        if k == "qkv":
            return {"bytes": e * S * D + w + 3 * tensor, "flops": proj}
        return {"bytes": 2 * e * S * D + w + e * D * H * d, "flops": proj + attn + 2 * S * D * H * d}
    return {"bytes": 4 * tensor, "flops": attn}


def draw(rng):
    """One more case: each kind as often as the others, lengths and widths spread over their
    logarithm, odd ones among them."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("forward", "slots", "attention", "train", "linear", "qkv", "layer"))
    dtype = rng.choice(("bf16", "bf16", "bf16", "fp32"))
    d = rng.choice((128, 128, 128, 64))
    # fp32 storage and heads of 64 are used at smaller sizes, and cost more for the same work.
    top = 8e12 if dtype == "bf16" and d == 128 else 1.5e12
    while True:
        case = dict(kind=kind, dtype=dtype)
        if kind == "linear":
            case.update(M=log(100, 60000), N=8 * log(16, 1920), K=64 * log(2, 80))
        else:
            H = rng.choice((1, 2, 3, 4, 5, 8, 10, 13, 20, 40))
            case.update(H=H, d=d)
            if kind in ("qkv", "layer"):
                grid = (rng.randint(1, 36), rng.randint(4, 40), rng.randint(4, 64))
                case.update(grid=",".join(map(str, grid)), D=64 * log(2, 80))
            else:
                case.update(S=log(200, 60000))
            if kind != "qkv":
                C = rng.randint(1, min(H, 4))
                case.update(chunks=",".join(str(H // C + (1 if c < H % C else 0)) for c in range(C)))
            if kind not in ("qkv", "attention"):
                S = _tokens(case)
                case.update(P=rng.choice([p for p in (1, 2, 3, 4, 8) if S % p == 0]))
            if kind == "train":
                # The workspace where it applies, in every other case.
                case.update(ds_heads=rng.choice((0, 1)) if dtype == "bf16" and d == 128 else 0)
        if work(case)["flops"] <= top and work(case)["bytes"] <= 4e9:
            return case


# ---------------------------------------------------------------------------
# Inputs and one pass
# ---------------------------------------------------------------------------
_context = None


def _ctx():
    """The scheduler context a program keeps."""
    global _context
    if _context is None:
        _context = hcms.Context(max_chunks=8)
    return _context


def _randn(g, shape, dtype, by=1.0):
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    return (x if by == 1.0 else x * by).to(DTYPES[dtype])


def _inputs(case, seed):
    """The case's input tensors, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt, k = case["dtype"], case["kind"]
    if k == "linear":
        K = case["K"]
        return dict(x=_randn(g, (case["M"], K), dt), w=_randn(g, (case["N"], K), dt, K ** -0.5))
    S, H, d = _tokens(case), case["H"], case["d"]
    if k in ("qkv", "layer"):
        D = case["D"]
        t = dict(x=_randn(g, (S, D), dt), w_qkv=_randn(g, (3 * H * d, D), dt, D ** -0.5))
        if k == "layer":
            t["w_o"] = _randn(g, (D, H * d), dt, (H * d) ** -0.5)
        return t
    shape = (H, S, d) if k == "attention" else (S, H, d)
    t = {n: _randn(g, shape, dt) for n in "qkv"}
    if k == "train":
        t["dout"] = _randn(g, shape, dt)
    return t


def prepare(case, seed):
    s = dict(case, t=_inputs(case, seed))
    k = case["kind"]
    if "d" in case:
        s["scale"] = case["d"] ** -0.5
    if "chunks" in case:
        s["sizes"] = _ints(case["chunks"])
    if "grid" in case:
        s["dims"] = _ints(case["grid"])
        s["pairs"] = _pairs(case["d"], len(s["dims"]))
        s["table"] = hcms.rope_table(s["dims"], s["pairs"], BASE)
    if k == "train":
        for n in "qkv":
            s["t"][n].requires_grad_(True)
        s["ctx"] = _ctx()
        if case["ds_heads"]:
            # Its own context, which holds the score-gradient workspace: two regions.
            s["ctx"] = hcms.Context(max_chunks=8)
            n = 2 * case["ds_heads"] * hcms.backward_ds_bytes(case["S"], case["d"])
            s["ctx"].set_ds_workspace(torch.empty(n, dtype=torch.uint8, device="cuda"))
    elif k in ("forward", "slots", "layer"):
        s["ctx"] = _ctx()
    return s


def run(s):
    t, k = s["t"], s["kind"]
    if k == "linear":
        return hcms.linear(t["x"], t["w"])
    if k == "qkv":
        return hcms.qkv_projection(t["x"], t["w_qkv"], s["H"], s["d"], s["table"], s["dims"],
                                   s["pairs"])
    if k == "attention":
        return hcms.attention(t["q"], t["k"], t["v"], s["scale"], s["sizes"])
    if k == "forward":
        return s["ctx"].forward(t["q"], t["k"], t["v"], s["P"], s["scale"], s["sizes"])
    if k == "slots":
        return s["ctx"].forward_slots(t["q"], t["k"], t["v"], s["P"], s["scale"], s["sizes"])
    if k == "layer":
        return s["ctx"].layer_forward(t["x"], t["w_qkv"], t["w_o"], s["P"], s["H"], s["d"],
                                      s["scale"], s["sizes"], s["table"], s["dims"], s["pairs"])
    out = hcms.HcmsAttention.apply(t["q"], t["k"], t["v"], s["ctx"], s["P"], s["scale"], s["sizes"])
    return (out.detach(), *torch.autograd.grad(out, (t["q"], t["k"], t["v"]), t["dout"]))


# ---------------------------------------------------------------------------
# Accuracy
# ---------------------------------------------------------------------------
def tolerance(case):
    # Four times the error against 64 bits: 1.7e-3 for a projection (its bf16 result's rounding),
    # 2.4e-3 where the softmax weights are rounded to bf16 too (3.2e-3 with fp32 storage, whose
    # inputs are rounded as well), up to 4.9e-3 for a whole layer.
    if case["kind"] in ("linear", "qkv"):
        return {"rel": 7e-3}
    if case["kind"] == "layer":
        return {"rel": 2e-2}
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 1.3e-2}


def _softmax_rows(q, k, scale):
    return torch.softmax((q @ k.T) * scale, dim=1)


def _attention64(q, k, v, scale, rows=4096):
    """Attention of one head, [S][d] in float64."""
    return torch.cat([_softmax_rows(x, k, scale) @ v for x in q.split(rows)])


def _train64(q, k, v, dout, scale, rows=4096):
    """Output and gradients of one head, [S][d] in float64."""
    out, dq, dk, dv = torch.empty_like(q), torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for i in range(0, q.shape[0], rows):
        r = slice(i, i + rows)
        p = _softmax_rows(q[r], k, scale)
        out[r] = p @ v
        dv += p.T @ dout[r]
        dp = dout[r] @ v.T
        ds = p * (dp - (p * dp).sum(1, keepdim=True)) * scale
        dq[r] = ds @ k
        dk += ds.T @ q[r]
    return out, dq, dk, dv


def _rotate64(x, grid, d):
    """The rotary embedding of [S][H][d] on a row-major grid: pair i of axis a's n pairs turns by
    the axis's coordinate times BASE^(-i / n)."""
    S = x.shape[0]
    rest = torch.arange(S, device=x.device)
    coords = []
    for n in reversed(grid):
        coords.insert(0, (rest % n).double())
        rest = rest // n
    angle = torch.cat([c[:, None] * BASE ** (-torch.arange(n, device=x.device).double() / n)
                       for c, n in zip(coords, _pairs(d, len(grid)))], dim=1)[:, None, :]
    a, b = x[..., 0::2], x[..., 1::2]
    cos, sin = angle.cos(), angle.sin()
    return torch.stack((a * cos - b * sin, a * sin + b * cos), dim=-1).reshape(x.shape)


def exact(case, seed):
    t = {n: x.double() for n, x in _inputs(case, seed).items()}
    k = case["kind"]
    if k == "linear":
        return t["x"] @ t["w"].T
    S, H, d = _tokens(case), case["H"], case["d"]
    scale = d ** -0.5
    if k == "attention":
        return torch.stack([_attention64(t["q"][h], t["k"][h], t["v"][h], scale) for h in range(H)])
    if k == "train":
        heads = [_train64(*(t[n][:, h].contiguous() for n in ("q", "k", "v", "dout")), scale)
                 for h in range(H)]
        return tuple(torch.stack(x, dim=1) for x in zip(*heads))
    if k in ("qkv", "layer"):
        grid = _ints(case["grid"])
        y = (t["x"] @ t["w_qkv"].T).reshape(S, 3, H, d)
        q, kk, v = _rotate64(y[:, 0], grid, d), _rotate64(y[:, 1], grid, d), y[:, 2]
        if k == "qkv":
            return q, kk, v
        t.update(q=q, k=kk, v=v)
    out = torch.stack([_attention64(*(t[n][:, h].contiguous() for n in "qkv"), scale)
                       for h in range(H)], dim=1)
    return out if k != "layer" else out.reshape(S, H * d) @ t["w_o"].T
