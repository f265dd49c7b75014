"""The calls by which this library's speed is measured, through its torch
binding: attention training steps, ring steps, attention blocks with their
projections, the projection product and the rotary embedding.

A case is a dict of plain values with a ``kind``:

  attn   forward and backward of the attention of one GPU's share of heads
  ring   one rank's ring attention over two key/value blocks: its own block
         (causal), the block before it (all keys visible), and the merge
  layer  forward and backward of the attention block with its projections
  gemm   the projection product on its own
  rope   rotary embedding in place: queries and keys forward, their gradients
         back, for callers that project Q and K themselves

``prepare`` makes what a training program holds before the call (inputs on
the GPU, the workspace it keeps from step to step), ``run`` is one pass, and
``exact`` is the same result from plain torch in 64 bits.
"""

import math

import torch

from paper_2602_21196_amd import upipe

D = 128                   # head width, the only one the library builds
DEV = "cuda:0"


# ------------------------------------------------------------------- cases

def listed():
    return [
        # A unit-test sized step: launches and latency are all there is.
        dict(name="attn_tiny", kind="attn", B=1, S=512, Hq=2, Hkv=1, U=1, causal=True),
        # A short document of odd length, two key/value groups cut by the chunks.
        dict(name="attn_ragged_4k", kind="attn", B=1, S=4100, Hq=8, Hkv=2, U=2, causal=True),
        # Bidirectional attention (an encoder) of a ragged length.
        dict(name="attn_bidir_2k", kind="attn", B=1, S=2500, Hq=4, Hkv=2, U=2, causal=False),
        # The batch-size ablation at a pre-training length: Llama3-8B share.
        dict(name="attn_batch_8k", kind="attn", B=4, S=8192, Hq=4, Hkv=1, U=1, causal=True),
        # Qwen3-32B share (8 query heads on one key/value head), two heads a chunk.
        dict(name="attn_qwen_32k", kind="attn", B=1, S=32768, Hq=8, Hkv=1, U=2, causal=True),
        # The long-context headline: Llama3-8B share at 128K tokens, one head a chunk.
        dict(name="attn_llama_128k", kind="attn", B=1, S=131072, Hq=4, Hkv=1, U=1, causal=True),
        # Ulysses + Ring hybrid: two ring steps of a 32K block and their merge.
        dict(name="ring_32k", kind="ring", S=32768, Skv=32768, Hq=4, Hkv=1, U=1),
        # The attention block of the Llama3-8B share at its pre-training length.
        dict(name="layer_llama_8k", kind="layer", B=1, S=8192, dm=4096, Hq=4, Hkv=1, U=1,
             rope=500000.0, full=False),
        # Short ragged sequences in a batch, attention output recomputed, no RoPE.
        dict(name="layer_batch_3k_full", kind="layer", B=2, S=3000, dm=2048, Hq=8, Hkv=2, U=4,
             rope=0.0, full=True),
        # Long-context block of the Qwen3-32B share.
        dict(name="layer_qwen_64k", kind="layer", B=1, S=65536, dm=5120, Hq=8, Hkv=1, U=1,
             rope=1000000.0, full=False),
        # A projection outside the block, at the Llama3-8B width.
        dict(name="gemm_8k", kind="gemm", M=8192, N=4096, K=4096),
        # Rotary embedding on its own at the headline length.
        dict(name="rope_128k", kind="rope", S=131072, Hq=4, Hkv=1, base=500000.0),
    ]


def _log_int(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _length(rng, lo, hi):
    """A sequence length: odd as often as a multiple of 128."""
    S = _log_int(rng, lo, hi)
    return max(lo, S // 128 * 128) if rng.random() < 0.5 else S


def _heads(rng):
    """(Hq, Hkv, U) of one GPU's share."""
    Hkv = rng.choice([1, 1, 1, 2])
    Hq = Hkv * rng.choice([1, 2, 4, 8] if Hkv == 1 else [2, 4])
    return Hq, Hkv, rng.choice([u for u in range(1, Hq + 1) if Hq % u == 0])


def draw(rng):
    cap = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["attn", "attn", "attn", "ring", "layer", "layer", "gemm", "rope"])
        Hq, Hkv, U = _heads(rng)
        if kind == "attn":
            c = dict(kind=kind, B=rng.choice([1, 1, 1, 2, 4]), S=_length(rng, 512, 131072), Hq=Hq,
                     Hkv=Hkv, U=U, causal=rng.random() < 0.8)
        elif kind == "ring":
            S = _length(rng, 1024, 32768)
            c = dict(kind=kind, S=S, Skv=rng.choice([S, _length(rng, 1024, 32768)]), Hq=Hq,
                     Hkv=Hkv, U=U)
        elif kind == "layer":
            c = dict(kind=kind, B=rng.choice([1, 1, 2]), S=_length(rng, 2048, 65536),
                     dm=rng.choice([2048, 4096, 5120]), Hq=Hq, Hkv=Hkv, U=U,
                     rope=rng.choice([0.0, 500000.0, 1000000.0]), full=rng.random() < 0.3)
        elif kind == "gemm":
            c = dict(kind=kind, M=128 * _log_int(rng, 4, 128), N=128 * _log_int(rng, 4, 40),
                     K=128 * _log_int(rng, 4, 64))
        else:
            c = dict(kind=kind, S=_length(rng, 1024, 131072), Hq=Hq, Hkv=Hkv,
                     base=rng.choice([10000.0, 500000.0, 1000000.0]))
        if work(c)["flops"] <= cap:
            return c


# --------------------------------------------------------- work, tolerance

def _pairs(S, causal):
    return S * (S + 1) // 2 if causal else S * S


def work(c):
    """Forward 4 d per visible (query, key, head) triple, backward 2.5 times
    that; 2 M N K per product.  The block's backward gets x and the weights
    only, so forming Q, K, V again belongs to it, and with full checkpointing
    the attention forward does too."""
    kind = c["kind"]
    if kind == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        return {"bytes": 2 * (M * K + K * N + M * N), "flops": 2 * M * N * K}
    S, Hq, Hkv = c["S"], c["Hq"], c["Hkv"]
    if kind == "rope":
        n = 2 * S * (Hq + Hkv) * D          # q, k and their gradients
        return {"bytes": 4 * n, "flops": 3 * n}
    if kind == "ring":
        Skv = c["Skv"]
        qo, kv = 2 * S * Hq * D, 2 * 2 * Hkv * D
        pairs = _pairs(S, True) + S * Skv
        return {"bytes": 2 * qo + kv * (S + Skv) + 4 * Hq * S, "flops": 4 * D * Hq * pairs}
    B = c["B"]
    heads, lse = 2 * B * S * D, 4 * B * Hq * S       # bytes of one head, of lse
    if kind == "attn":
        fwd = 4 * D * Hq * B * _pairs(S, c["causal"])
        # q, do in; o, dq out; k, v in; dk, dv out; lse
        return {"bytes": heads * (4 * Hq + 4 * Hkv) + lse, "flops": int(3.5 * fwd)}
    dm = c["dm"]
    fwd = 4 * D * Hq * B * _pairs(S, True)
    attn = (4.5 if c["full"] else 3.5) * fwd
    qkv, proj = 2 * B * S * dm * (Hq + 2 * Hkv) * D, 2 * B * S * dm * Hq * D
    # forward QKV, y; backward QKV again, dFO, dWo, dX, dWqkv
    w = 2 * dm * (2 * Hq + 2 * Hkv) * D
    return {"bytes": 2 * B * S * dm * 4 + 2 * w + heads * Hq + lse,
            "flops": int(attn + 4 * qkv + 3 * proj)}


def tolerance(c):
    """Outputs are bf16 (lse fp32) from bf16 inputs with fp32 sums; P and dS
    (in the block Q, K, V, O and their gradients too) are rounded to bf16
    inside.  About four times the distance from `exact` over these ranges:
    rel 1.7e-3 (gemm, rope), 3.4e-3 (ring: two roundings of o), 2.5e-3 (attn),
    5.5e-3 (layer); max 4e-3, 2.4e-2, 0.19 and 0.34 -- the gradients of the
    first rows and keys are far above the root mean square of a long
    sequence, and so are their roundings."""
    kind = c["kind"]
    if kind in ("gemm", "rope"):
        return {"rel": 6e-3, "max": 1.6e-2}
    if kind == "ring":
        return {"rel": 1.3e-2, "max": 1e-1}
    if kind == "attn":
        return {"rel": 1e-2, "max": 7e-1}
    return {"rel": 2e-2, "max": 1.0}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _draw(g, shape, std=1.0):
    t = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)
    return t.mul_(std).to(torch.bfloat16)


def _inputs(c, seed):
    """The case's input tensors: activations N(0, 1), weights N(0, 0.02^2)."""
    g = _gen(seed)
    kind = c["kind"]
    if kind == "gemm":
        return dict(a=_draw(g, (c["M"], c["K"])), b=_draw(g, (c["K"], c["N"]), 0.02))
    S, Hq, Hkv = c["S"], c["Hq"], c["Hkv"]
    if kind == "rope":
        return dict(q=_draw(g, (S, Hq, D)), k=_draw(g, (S, Hkv, D)),
                    dq=_draw(g, (S, Hq, D)), dk=_draw(g, (S, Hkv, D)))
    if kind == "ring":
        n = c["Skv"]
        return dict(q=_draw(g, (S, Hq, D)), k=_draw(g, (S, Hkv, D)), v=_draw(g, (S, Hkv, D)),
                    k0=_draw(g, (n, Hkv, D)), v0=_draw(g, (n, Hkv, D)))
    lead = (c["B"], S) if c["B"] > 1 else (S,)
    if kind == "attn":
        return dict(q=_draw(g, lead + (Hq, D)), k=_draw(g, lead + (Hkv, D)),
                    v=_draw(g, lead + (Hkv, D)), do=_draw(g, lead + (Hq, D)))
    dm = c["dm"]
    return dict(x=_draw(g, lead + (dm,)), wqkv=_draw(g, (dm, (Hq + 2 * Hkv) * D), 0.02),
                wo=_draw(g, (Hq * D, dm), 0.02), dy=_draw(g, lead + (dm,)))


def prepare(c, seed):
    s = dict(c, **_inputs(c, seed))
    kind = c["kind"]
    need = 0
    if kind == "attn":
        a = (c["S"], c["Hq"], c["Hkv"], D, c["U"])
        need = max(upipe.upipe_attn_fwd_workspace_size(*a), upipe.upipe_attn_bwd_workspace_size(*a))
    elif kind == "ring":
        a = (c["Hq"], c["Hkv"], D, c["U"])
        need = max(upipe.upipe_attn_fwd_ring_workspace_size(c["S"], n, *a)
                   for n in (c["S"], c["Skv"]))
    elif kind == "layer":
        a = (c["S"], c["dm"], c["Hq"], c["Hkv"], D, c["U"])
        need = max(upipe.upipe_layer_fwd_workspace_size(*a),
                   upipe.upipe_layer_bwd_workspace_size(*a))
    if need:
        s["ws"] = upipe.workspace(need, DEV)
    return s


def run(s):
    kind = s["kind"]
    if kind == "gemm":
        return upipe.gemm(s["a"], s["b"])
    if kind == "rope":
        base = s["base"]
        return (upipe.rope(s["q"], base), upipe.rope(s["k"], base),
                upipe.rope(s["dq"], base, inverse=True), upipe.rope(s["dk"], base, inverse=True))
    U, ws = s["U"], s["ws"]
    if kind == "ring":
        off = s["Skv"]         # the rank's block follows the other one
        o, lse = upipe.attn_fwd_ring(s["q"], s["k"], s["v"], off, off, U=U, ws=ws)
        o0, lse0 = upipe.attn_fwd_ring(s["q"], s["k0"], s["v0"], off, 0, U=U, ws=ws)
        return upipe.lse_merge(o, lse, o0, lse0)
    if kind == "attn":
        causal = s["causal"]
        o, lse = upipe.attn_fwd(s["q"], s["k"], s["v"], causal=causal, U=U, ws=ws)
        return (o, lse) + tuple(upipe.attn_bwd(s["q"], s["k"], s["v"], o, lse, s["do"],
                                               causal=causal, U=U, ws=ws))
    heads = dict(U=U, ws=ws, rope_base=s["rope"])
    y, o, lse = upipe.layer_fwd(s["x"], s["wqkv"], s["wo"], s["Hq"], s["Hkv"], **heads)
    kept = (None, None) if s["full"] else (o, lse)
    g = upipe.layer_bwd(s["x"], s["wqkv"], s["wo"], *kept, s["dy"], s["Hq"], s["Hkv"], **heads)
    return (y, o, lse) + tuple(g)


# ------------------------------------------------- the same in 64 bits

ROWS = 1024               # query rows formed at a time


def _attn64(q, k, v, do, delta, causal):
    """One sequence in float64: o, lse and, with do, dq, dk, dv.  Query i sees
    key j iff j <= i + delta (every key without causal)."""
    S, Hq, _ = q.shape
    n, Hkv, _ = k.shape
    G = Hq // Hkv
    scale = 1.0 / math.sqrt(D)
    o = torch.zeros_like(q)
    lse = torch.empty((Hq, S), dtype=torch.float64, device=q.device)
    dq = torch.zeros_like(q) if do is not None else None
    dk, dv = (torch.zeros_like(k), torch.zeros_like(v)) if do is not None else (None, None)
    for h in range(Hq):
        g = h // G
        kh, vh = k[:, g].contiguous(), v[:, g].contiguous()
        for r0 in range(0, S, ROWS):
            r1 = min(S, r0 + ROWS)
            e = min(n, r1 + delta) if causal else n
            qh = q[r0:r1, h].contiguous()
            s = (qh @ kh[:e].t()).mul_(scale)
            if causal and r0 + delta < e - 1:
                row = torch.arange(r0, r1, device=q.device).unsqueeze(1) + delta
                s.masked_fill_(torch.arange(e, device=q.device) > row, -math.inf)
            L = torch.logsumexp(s, dim=1)
            p = s.sub_(L.unsqueeze(1)).exp_()
            oh = p @ vh[:e]
            o[r0:r1, h], lse[h, r0:r1] = oh, L
            if do is not None:
                dh = do[r0:r1, h].contiguous()
                dv[:e, g] += p.t() @ dh
                ds = (dh @ vh[:e].t()).sub_((dh * oh).sum(1, keepdim=True)).mul_(p).mul_(scale)
                dq[r0:r1, h] = ds @ kh[:e]
                dk[:e, g] += ds.t() @ qh
    return (o, lse) if do is None else (o, lse, dq, dk, dv)


def _rope64(x, base, sign=1.0):
    """Pair (e, e + 64) of row s turned by the angle s base^(-e/64)."""
    e = torch.arange(D // 2, dtype=torch.float64, device=x.device)
    ang = torch.arange(x.shape[0], dtype=torch.float64, device=x.device).unsqueeze(1) * \
        torch.exp(-e / (D // 2) * math.log(base))
    cos, sin = ang.cos().unsqueeze(1), sign * ang.sin().unsqueeze(1)
    a, b = x[..., :D // 2], x[..., D // 2:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1)


def _layer64(x, wqkv, wo, dy, Hq, Hkv, base):
    S = x.shape[0]
    qkv = (x @ wqkv).view(S, Hq + 2 * Hkv, D)
    q, k, v = qkv[:, :Hq], qkv[:, Hq:Hq + Hkv], qkv[:, Hq + Hkv:]
    if base:
        q, k = _rope64(q, base), _rope64(k, base)
    do = (dy @ wo.t()).view(S, Hq, D)
    o, lse, dq, dk, dv = _attn64(q.contiguous(), k.contiguous(), v.contiguous(), do, 0, True)
    if base:
        dq, dk = _rope64(dq, base, -1.0), _rope64(dk, base, -1.0)
    dqkv = torch.cat([dq, dk, dv], dim=1).view(S, -1)
    of = o.view(S, Hq * D)
    return of @ wo, o, lse, dqkv @ wqkv.t(), x.t() @ dqkv, of.t() @ dy


def exact(c, seed):
    kind = c["kind"]
    if kind == "layer" and work(c)["flops"] > 2e13:
        return None           # over 20 seconds in 64 bits
    t = {n: x.double() for n, x in _inputs(c, seed).items()}
    if kind == "gemm":
        return t["a"] @ t["b"]
    if kind == "rope":
        return (_rope64(t["q"], c["base"]), _rope64(t["k"], c["base"]),
                _rope64(t["dq"], c["base"], -1.0), _rope64(t["dk"], c["base"], -1.0))
    if kind == "ring":
        n = c["Skv"]
        k, v = torch.cat([t["k0"], t["k"]]), torch.cat([t["v0"], t["v"]])
        return _attn64(t["q"], k, v, None, n, True)
    if kind == "attn":
        seqs = [(t["q"], t["k"], t["v"], t["do"])] if c["B"] == 1 else \
            list(zip(t["q"], t["k"], t["v"], t["do"]))
        outs = [_attn64(*s, 0, c["causal"]) for s in seqs]
        return outs[0] if c["B"] == 1 else tuple(torch.stack(z) for z in zip(*outs))
    seqs = [(t["x"], t["dy"])] if c["B"] == 1 else list(zip(t["x"], t["dy"]))
    outs = [_layer64(x, t["wqkv"], t["wo"], dy, c["Hq"], c["Hkv"], c["rope"]) for x, dy in seqs]
    if c["B"] == 1:
        return outs[0]
    z = list(zip(*outs))
    return tuple(torch.stack(a) for a in z[:4]) + tuple(sum(a) for a in z[4:])
