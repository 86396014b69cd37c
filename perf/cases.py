"""The calls whose speed matters: sizes, inputs, one pass through the public
entry points, the work a pass cannot do without, and a 64-bit reference.

A case names a path (`kind`) of the package and its sizes:
  forward    hla.forward, masked or unmasked, normalised or not, bf16 or fp32
  decay      hla.forward_decay
  ahla       hla.ahla_forward
  hla3       hla.hla3_forward
  train      hla.hla2_attention and its gradients (bf16), as a training step takes them
  backward   hla.backward (fp32 gradients)
  prefill    a new hla.State and hla.prefill over the prompt, `piece` tokens a call
  step       hla.step on a state that has read `n` tokens

Inputs: q and k rows of unit length and v ~ N(0,1) in bf16; N(0,1)/sqrt(d) in
fp32.  Where the output is normalised q and k are non-negative (a positive
feature map, which a ratio needs: with signed rows the denominator crosses 0).
"""
import torch

import paper_2510_27258_amd as hla

EPS = 1e-6
DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}


def _case(kind, B, H, n, d, chunk, dtype="bf16", masked=True, normalized=False, **more):
    return dict(kind=kind, B=B, H=H, n=n, d=d, chunk=chunk, dtype=dtype, masked=masked, normalized=normalized, **more)


def listed():
    return [
        # the smallest call: a short sequence in fp32, where launches and latency count
        dict(_case("forward", 1, 2, 256, 32, 64, "fp32"), name="forward-fp32-small"),
        # a layer of a d = 64 model over a training batch
        dict(_case("forward", 4, 16, 4096, 64, 64), name="forward-d64"),
        # a layer of a d = 128 model over long normalised sequences, the benchmark's workload and the largest case
        dict(_case("forward", 2, 32, 16384, 128, 128, normalized=True), name="forward-d128-norm"),
        # fp32 activations: evaluation and gradient checks of the d = 64 layer
        dict(_case("forward", 2, 16, 4096, 64, 64, "fp32"), name="forward-fp32"),
        # the unmasked operator, normalised by its row sums, over a ragged length
        dict(_case("forward", 1, 16, 4001, 128, 128, masked=False, normalized=True), name="forward-unmasked"),
        # a layer with exponential decay
        dict(_case("decay", 4, 16, 4096, 64, 64, gamma=0.99), name="decay-d64"),
        # the asymmetric variant at d = 128, ragged length
        dict(_case("ahla", 2, 32, 8000, 128, 128), name="ahla-d128"),
        # the third-order operator in fp32
        dict(_case("hla3", 1, 8, 2048, 16, 32, "fp32"), name="hla3-fp32"),
        # a training step's layer: forward and gradients through autograd
        dict(_case("train", 4, 16, 4096, 64, 64), name="train-d64"),
        # the gradients alone at d = 128, few heads and a long sequence
        dict(_case("backward", 1, 8, 16384, 128, 64), name="backward-d128"),
        # serving: a prompt of ragged length read in two calls
        dict(_case("prefill", 1, 32, 8000, 128, 128, piece=4096), name="prefill-d128"),
        # serving: one token for each of 64 sequences of a 32-head layer
        dict(_case("step", 64, 32, 256, 128, 128), name="step-d128"),
    ]


# kind -> (largest B*H*n*d of a drawn case, dtypes, d, chunks)
_RANGES = {
    "forward": (1 << 26, ("bf16",), (32, 64, 128), (64, 128)),
    "forward-fp32": (1 << 23, ("fp32",), (32, 64, 128), (32, 64, 128)),
    "forward-unmasked": (1 << 23, ("bf16", "fp32"), (32, 64, 128), (64, 128)),
    "decay": (1 << 25, ("bf16",), (64, 128), (64, 128)),
    "ahla": (1 << 25, ("bf16",), (64, 128), (64, 128)),
    "hla3": (1 << 20, ("fp32", "bf16"), (16, 32), (32, 64)),
    "train": (1 << 24, ("bf16",), (64, 128), (64, 128)),
    "backward": (1 << 24, ("bf16",), (64, 128), (64, 128)),
    "prefill": (1 << 25, ("bf16",), (64, 128), (64, 128)),
    "step": (1 << 25, ("bf16", "fp32"), (64, 128), (64,)),
}


def draw(rng):
    path = rng.choice(sorted(_RANGES))
    most, dtypes, ds, chunks = _RANGES[path]
    kind = path.split("-")[0]
    d, dtype, chunk = rng.choice(ds), rng.choice(dtypes), rng.choice(chunks)
    if kind == "step":
        B, H = round(2 ** rng.uniform(0, 6)), rng.choice((4, 8, 12, 16, 32))
        return _case(kind, B, H, rng.randint(1, 256 * 64 // (B * H) + 8), d, chunk, dtype, masked=rng.random() < 0.8)
    B, H = rng.choice((1, 1, 2, 3, 4)), rng.choice((1, 2, 5, 8, 12, 16, 32))
    top = min(most // (B * H * d), 32768)
    low = min(100, top // 2)
    n = min(top, round(low * (top / low) ** rng.random()))
    c = _case(kind, B, H, n, d, chunk, dtype)
    if path == "forward-unmasked":
        c["masked"] = False
    if kind in ("forward", "decay", "ahla", "hla3", "prefill"):
        c["normalized"] = rng.random() < 0.4
    if kind == "hla3":
        c["masked"] = rng.random() < 0.6
    if kind == "decay":
        c["gamma"] = rng.choice((0.9, 0.97, 0.99, 0.999))
    if kind == "prefill":
        c["piece"] = rng.choice((1024, 2048, 4096, 8192))
    return c


def _tokens(g, c, n):
    B, H, d = c["B"], c["H"], c["d"]
    q, k, v = (torch.randn(B, H, n, d, generator=g, device="cuda") for _ in range(3))
    if c["normalized"]:
        q, k = q.abs(), k.abs()
    if c["dtype"] == "fp32":
        return q * d ** -0.5, k * d ** -0.5, v * d ** -0.5
    q, k = (x / x.norm(dim=-1, keepdim=True) for x in (q, k))
    return q.bfloat16(), k.bfloat16(), v.bfloat16()


def _inputs(case, seed):
    """Everything that is drawn, made from the seed alone."""
    g = torch.Generator("cuda").manual_seed(seed)
    s = dict(case=case)
    s["q"], s["k"], s["v"] = _tokens(g, case, case["n"])
    if case["kind"] in ("train", "backward"):
        s["g"] = torch.randn(s["v"].shape, generator=g, device="cuda")
    if case["kind"] == "step":
        s["tok"] = tuple(x[:, :, 0].contiguous() for x in _tokens(g, case, 1))
    return s


def _state(c):
    return hla.State(c["B"], c["H"], c["d"], c["d"], masked=c["masked"], normalized=c["normalized"], eps=EPS,
                     dtype=DTYPES[c["dtype"]])


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "train":
        for x in "qkv":
            s[x].requires_grad_()
    if case["kind"] == "prefill":
        cuts = range(0, case["n"], case["piece"])
        s["pieces"] = [tuple(s[x][:, :, i:i + case["piece"]].contiguous() for x in "qkv") for i in cuts]
        del s["q"], s["k"], s["v"]
    if case["kind"] == "step":
        s["state"] = _state(case)
        hla.prefill(s["state"], s["q"], s["k"], s["v"], case["chunk"], want_out=False)
        del s["q"], s["k"], s["v"]
    return s


def run(s):
    c = s["case"]
    kind, chunk, how = c["kind"], c["chunk"], dict(normalized=c["normalized"], eps=EPS)
    if kind == "forward":
        # the automatic choice sizes its workspace for the masked operator; the unmasked one names its algorithm
        algo = hla.capi.HLA_ALGO_AUTO if c["masked"] else hla.capi.HLA_ALGO_CHUNKED
        return hla.forward(s["q"], s["k"], s["v"], chunk, masked=c["masked"], algo=algo, **how)
    if kind == "decay":
        return hla.forward_decay(s["q"], s["k"], s["v"], chunk, c["gamma"], masked=c["masked"], **how)
    if kind == "ahla":
        return hla.ahla_forward(s["q"], s["k"], s["v"], chunk, **how)
    if kind == "hla3":
        return hla.hla3_forward(s["q"], s["k"], s["v"], chunk, masked=c["masked"], **how)
    if kind == "train":
        out = hla.hla2_attention(s["q"], s["k"], s["v"], chunk)
        return [out.detach(), *torch.autograd.grad(out, (s["q"], s["k"], s["v"]), s["g"])]
    if kind == "backward":
        return list(hla.backward(s["q"], s["k"], s["v"], s["g"], chunk))
    if kind == "prefill":
        state = _state(c)
        outs = [hla.prefill(state, q, k, v, chunk) for q, k, v in s["pieces"]]
        return [*outs, state.data]
    return [hla.step(s["state"], *s["tok"]), s["state"].data]


def work(case):
    """Bytes: inputs and outputs once.  Flops: the serial recurrence's (the
    state updates and the readout of one token, no chunking)."""
    d, kind = case["d"], case["kind"]
    es = 2 if case["dtype"] == "bf16" else 4
    rows = case["B"] * case["H"] * (1 if kind == "step" else case["n"])
    record = case["B"] * case["H"] * (d * (d + 1) // 2 + 2 * d * d + 2 * d) * 4
    tokens = rows * 3 * d * es
    out = rows * d * 4
    per = {"ahla": 8, "hla3": 20, "train": 14 + 34, "backward": 34}.get(kind, 14)
    moved = {"train": 3 * tokens + 2 * out, "backward": tokens + 4 * out, "prefill": tokens + out + record,
             "step": tokens + out + 2 * record}.get(kind, tokens + out)
    return {"bytes": moved, "flops": rows * per * d * d}


def tolerance(case):
    """About four times the distance to the 64-bit sums that these paths show."""
    if case["kind"] == "train":
        return {"rel": 4e-3, "max": 2e-2}     # gradients rounded to bf16
    if case["kind"] == "step":
        return {"rel": 1.2e-5}                # the state comes from a bf16 prompt
    if case["dtype"] == "fp32" or not case["masked"] or case["kind"] == "hla3":
        return {"rel": 2.5e-6}                # up to 6e-7 seen
    return {"rel": 2.5e-5}                    # computed operands carry 16 bits: up to 6e-6 seen


def _exact_head(c, q, k, v, g):
    """(num, den, extra) of one head in 64 bits, by the dense sums."""
    n = q.shape[0]
    kind = c["kind"]
    one = torch.ones(n, 1, dtype=q.dtype, device=q.device)
    v1 = torch.cat([v, one], 1) if c["normalized"] else v
    W = (q @ k.T).tril_()
    if kind == "ahla":
        o = W @ (W @ v1)
    elif kind == "hla3" and c["masked"]:
        # triples (i, u, j) whose largest index is attained at least twice, by the token it falls on
        delta = W.diagonal().clone()[:, None]
        Ws = W.tril(-1)
        R = Ws @ k
        sigma = ((k @ q.T).tril_(-1) ** 2).sum(1, keepdim=True)
        X = (sigma + delta ** 2) * v1 + delta * (Ws @ v1)
        o = (q @ R.T).tril_() @ (delta * v1) + W @ X
    elif kind == "hla3":
        R = (W @ k @ q.T).tril_() @ q
        o = (R @ k.T).tril_() @ v1
    else:
        if kind == "decay":
            t = torch.arange(n, dtype=q.dtype, device=q.device)
            W *= (c["gamma"] ** (t[:, None] - t[None, :]).clamp_(min=0))
        R = W @ k
        T = (q @ R.T) if c["masked"] else (R @ q.T)
        if kind == "decay":
            T *= (c["gamma"] ** ((2 if c["masked"] else 1) * (t[:, None] - t[None, :]).clamp_(min=0)))
        o = T.tril_() @ v1
    if g is None:
        grads = None
    else:
        del T
        u = (v @ g.T).triu_() @ q
        dq = (g @ v.T).tril_() @ R + (u @ k.T).tril_() @ k
        dk = (k @ q.T).triu_() @ u + (k @ u.T).triu_() @ q
        grads = dq, dk, (R @ q.T).triu_() @ g
    num = o[:, :-1] / (o[:, -1:] + EPS) if c["normalized"] else o
    return num, grads


def _exact_state(q, k, v):
    """Packed records [heads, FP] after the tokens q, k, v [heads, n, d]."""
    d = q.shape[-1]
    A = (k @ q.transpose(1, 2).contiguous()).tril_(-1)
    kt = k.transpose(1, 2).contiguous()
    S, C = kt @ k, q.transpose(1, 2).contiguous() @ v
    G, h = kt @ (A @ v), (kt @ A.sum(2, keepdim=True))[:, :, 0]
    # S's upper triangle as d/2 pairs of rows p and d-1-p
    fold = [(a, j) for p in range(d // 2) for a in (p, d - 1 - p) for j in range(a, d)]
    rows, cols = torch.tensor(fold, device=q.device).unbind(1)
    return torch.cat([S[:, rows, cols], C.flatten(1), q.sum(1), G.flatten(1), h], 1)


def exact(case, seed):
    s = _inputs(case, seed)
    c, B, H, n, d = case, case["B"], case["H"], case["n"], case["d"]
    if c["kind"] == "step":
        q, k, v = (torch.cat([s[x], t[:, :, None]], 2).double().flatten(0, 1) for x, t in zip("qkv", s["tok"]))
        rec = torch.cat([_exact_state(q[i:i + 256], k[i:i + 256], v[i:i + 256]) for i in range(0, B * H, 256)])
        r = torch.tril(q @ k.transpose(1, 2).contiguous()) @ k
        t = r @ q[:, -1, :, None] if c["masked"] else q @ r[:, -1, :, None]
        o = t.transpose(1, 2).contiguous() @ v
        return [o[:, 0].reshape(B, H, d), rec.reshape(B, H, -1)]
    q, k, v = (s[x].flatten(0, 1) for x in "qkv")
    g = s["g"].flatten(0, 1) if "g" in s else None
    out = torch.empty(B * H, n, d, dtype=torch.float64, device="cuda")
    grads = [torch.empty_like(out) for _ in range(3)] if g is not None else []
    for i in range(B * H):
        out[i], got = _exact_head(c, q[i].double(), k[i].double(), v[i].double(), g[i].double() if g is not None else None)
        for to, x in zip(grads, got or ()):
            to[i] = x
    out, grads = out.reshape(B, H, n, d), [x.reshape(B, H, n, d) for x in grads]
    if c["kind"] == "train":
        return [out, *grads]
    if c["kind"] == "backward":
        return grads
    if c["kind"] == "prefill":
        rec = torch.cat([_exact_state(q[i:i + 1].double(), k[i:i + 1].double(), v[i:i + 1].double()) for i in range(B * H)])
        return [*(x.contiguous() for x in out.split(c["piece"], 2)), rec.reshape(B, H, -1)]
    return out
