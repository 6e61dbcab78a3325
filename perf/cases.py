"""The work a user of this library has it do, as cases that can be timed and compared.

Three kinds of case, each through a public entry point of the package:

  call         one invocation of a decoder: rs_decode_step (one new token for each of n sequences) or
               rs_catchup_prefill (spans of tokens the model has not seen), on a cache that already holds the
               sequences' contexts, with the fused entropy router behind the LM head.  Calls go to one stream that the
               program keeps, with buffers at fixed addresses, as the package's own host loop makes them.
  route        rs_route on logits a program already has
  router_plus  the learned router on hidden states

Shapes are those of the package's workloads (1.5B, 7B, 14B and 32B widths and the tiny pair); most cases run a few
layers of a shape, which is what the cost of a call is made of, and two run the whole 1.5B and 7B models.
Weights are N(0, 0.02) in bf16, caches hold N(0, 1) rows (the magnitude such weights produce), logit scales
lie in 0.5 .. 8, so the entropies the router sees cover its range.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import torch

import paper_2507_17307_amd as P

# name: layers of the whole model, d_model, query heads, KV heads, head_dim, d_ffn, tied LM head
SHAPES = {
    "tiny_s": (2, 128, 4, 2, 32, 384, True),
    "tiny_l": (4, 256, 8, 2, 32, 768, False),
    "s15": (28, 1536, 12, 2, 128, 8960, True),
    "m7": (28, 3584, 28, 4, 128, 18944, False),
    "m14": (48, 5120, 40, 8, 128, 13824, False),
    "m32": (64, 5120, 40, 8, 128, 27648, False),
}
VOCAB = 152064
EPS, THETA = 1e-6, 1e6
TAU = 0.8
ACTIVE = {"tiny_s": P.RS_SLM, "s15": P.RS_SLM}          # the small models of the pairs; the others are the large ones


def _call(name, shape, layers, seqs, rows, ctx_lo, ctx_hi, max_ctx, sample=False, vocab=VOCAB):
    """rows == seqs: a decode step; more: a catch-up.  Sequences hold ctx_lo .. ctx_hi positions before the call."""
    c = {"kind": "call", "shape": shape, "layers": layers, "vocab": vocab, "seqs": seqs, "rows": rows,
         "ctx_lo": ctx_lo, "ctx_hi": ctx_hi, "max_ctx": max_ctx, "sample": sample}
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # the router alone: one row of a small vocabulary (latency only), and a large batch of full rows
        {"name": "route_1x1024", "kind": "route", "n": 1, "vocab": 1024},
        {"name": "route_64x152064", "kind": "route", "n": 64, "vocab": VOCAB},
        # the learned router after a single-sequence step of the small model
        {"name": "router_plus_1", "kind": "router_plus", "n": 1, "d": 1536, "r": 8},
        # the two decode steps the stitched loop at batch 1 is made of: the whole small and the whole large model near
        # the end of a 4608-position cache
        _call("s15_decode_1", "s15", 28, 1, 1, 4570, 4570, 4608),
        _call("m7_decode_1", "m7", 28, 1, 1, 4561, 4561, 4608),
        # the loop's catch-ups after a switch: two rows on the small model, five on the large one
        _call("s15_catchup_2", "s15", 8, 1, 2, 2301, 2301, 4608),
        _call("m7_catchup_5", "m7", 6, 1, 5, 3107, 3107, 4608),
        # batched decode with sampling: 16 sequences of different lengths
        _call("m7_decode_16_sampled", "m7", 4, 16, 16, 512, 2047, 2048, sample=True),
        # the last chunk of a 2048-token prompt's prefill: the largest span one call takes
        _call("m7_prefill_128", "m7", 4, 1, 128, 1920, 1920, 4608),
        # a long catch-up late in a long context on the 14B width, an odd number of rows
        _call("m14_catchup_61", "m14", 4, 1, 61, 9001, 9001, 9216),
        # eight sequences with routing of their own on the 32B width: ragged spans in one call
        _call("m32_ragged_8", "m32", 3, 8, 29, 1200, 9900, 10240),
        # the largest batch: 128 sequences decode together
        _call("m7_decode_128", "m7", 4, 128, 128, 520, 1000, 1024),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    u = rng.random()
    if u < 0.15:
        return {"kind": "route", "n": _log_int(rng, 1, 128), "vocab": _log_int(rng, 64, 200000)}
    if u < 0.22:
        return {"kind": "router_plus", "n": _log_int(rng, 1, 128), "d": rng.choice([1536, 2048, 3584, 5120]),
                "r": rng.choice([8, 16, 32, 64])}
    shape = rng.choice(["s15"] * 5 + ["m7"] * 6 + ["m14"] * 4 + ["m32"] * 3 + ["tiny_s", "tiny_l"])
    layers = SHAPES[shape][0] if shape.startswith("tiny") else rng.randint(1, 3 if shape == "m32" else 4)
    if rng.random() < 0.4:
        seqs = rows = _log_int(rng, 1, 128)
    else:
        rows = _log_int(rng, 2, 128)
        seqs = min(_log_int(rng, 1, 16), rows - 1)
    # at most ~270 MB of cache per tensor: many sequences have shorter ones
    _, _, _, n_kv, hd, _, _ = SHAPES[shape]
    cap = (270 << 20) // (layers * seqs * n_kv * hd * 2)
    max_ctx = _log_int(rng, 512, max(600, min(10240, cap))) // 8 * 8
    span = rows - seqs + 1
    ctx_hi = rng.randint(max(200, max_ctx // 4), max_ctx - span)
    ctx_lo = rng.randint(200, ctx_hi) if seqs > 1 else ctx_hi
    return _call(None, shape, layers, seqs, rows, ctx_lo, ctx_hi, max_ctx, sample=rng.random() < 0.2,
                 vocab=rng.choice([VOCAB, VOCAB, VOCAB, 50257, 8192, rng.randint(1000, 32000)]))


# ------------------------------------------------------------------ layout of a call, from the case alone
def _spans(c):
    """(rows of every sequence, context of every sequence): ragged where there are several."""
    n, rows = c["seqs"], c["rows"]
    span = [1] * n
    for i in range(rows - n):                            # the spare rows go to sequences in an uneven pattern
        span[(i * i + i // 3) % n] += 1
    lo, hi = c["ctx_lo"], c["ctx_hi"]
    ctx = [lo + (i * 7919 + 13 * i * i) % (hi - lo + 1) for i in range(n)]
    return span, [min(x, c["max_ctx"] - s) for x, s in zip(ctx, span)]


def _slots(n):
    """KV slot of every sequence: all of them, in an order of its own."""
    step = next(s for s in (7, 5, 3, 11, 13) if math.gcd(s, n) == 1) if n > 1 else 1
    return [(i * step + n // 2) % n for i in range(n)]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, std, mean=0.0, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=g)


def _call_inputs(c, seed):
    """Weights, caches and call arguments on the GPU; the same for prepare() and exact()."""
    _, d, nq, nkv, hd, ffn, tied = SHAPES[c["shape"]]
    n_l, n, V, mc = c["layers"], c["seqs"], c["vocab"], c["max_ctx"]
    g = _gen(seed)
    w = SimpleNamespace(shape=SimpleNamespace(n_layers=n_l, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ffn=ffn,
                                              vocab=V, tied_lm_head=tied, rms_eps=EPS, rope_theta=THETA))
    w.embed = _normal(g, (V, d), 0.02)
    w.lm_head = w.embed if tied else _normal(g, (V, d), 0.02)
    w.final_norm = _normal(g, (d,), 0.05, 1.0)
    w.layers = [SimpleNamespace(attn_norm=_normal(g, (d,), 0.05, 1.0), w_qkv=_normal(g, ((nq + 2 * nkv) * hd, d), 0.02),
                                w_o=_normal(g, (d, nq * hd), 0.02), mlp_norm=_normal(g, (d,), 0.05, 1.0),
                                w_gate_up=_normal(g, (2 * ffn, d), 0.02), w_down=_normal(g, (d, ffn), 0.02))
                for _ in range(n_l)]
    k = _normal(g, (n_l, n, nkv, mc, hd), 1.0)           # [layer][slot][KV head][position][channel]
    v = _normal(g, (n_l, n, nkv, hd, mc), 1.0)           # transposed, as the library keeps it
    tok = torch.randint(0, V, (c["rows"],), device="cuda", generator=g).to(torch.int32)
    scale = torch.empty(n, device="cuda").uniform_(0.5, 8.0, generator=g)
    return w, k, v, tok, scale


_STREAM = []


def _stream():
    """The one stream the program makes its decoder calls on."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


# ------------------------------------------------------------------ prepare / run
def prepare(case, seed):
    c = case
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")  # noqa: E731
    if c["kind"] == "route":
        g = _gen(seed)
        n, V = c["n"], c["vocab"]
        s = SimpleNamespace(c=c, logits=_normal(g, (n, V), 1.2, dtype=torch.float32),
                            scale=torch.empty(n, device="cuda").uniform_(0.5, 8.0, generator=g), out=P.binding.new_route_out(n),
                            scratch=torch.empty(P.rs_route_scratch_bytes(n, V), dtype=torch.uint8, device="cuda"))
        return s
    if c["kind"] == "router_plus":
        hidden, w = _router_inputs(c, seed)
        n = c["n"]
        out = P.binding.new_route_out(n)
        out[:, 1] = 1 | 4                                # records of small-model steps above tau: the ones the router decides
        return SimpleNamespace(c=c, hidden=hidden, router=P.binding.RouterPlus(w), out=out, logits=torch.zeros(n, 2, device="cuda"))
    w, k, v, tok, scale = _call_inputs(c, seed)
    n = c["seqs"]
    m = P.Model(w, c["max_ctx"], max_seqs=n, max_rows=c["rows"])
    m.kv_k.copy_(k.view(-1))
    m.kv_v.copy_(v.view(-1))
    if c["sample"]:
        P.binding.rs_set_sampling(m.handle, True, 0x5EED0000 + seed)
    span, ctx = _spans(c)
    off = [0]
    for x in span:
        off.append(off[-1] + x)
    s = SimpleNamespace(c=c, m=m, slot=i32(_slots(n)), tok=tok, off=i32(off), pos=i32(ctx), scale=scale,
                        out=P.binding.new_route_out(n), logits=torch.zeros(n, c["vocab"], device="cuda"),
                        k=m.kv_k.view(k.shape), v=m.kv_v.view(v.shape), stream=_stream(), active=ACTIVE.get(c["shape"], P.RS_LLM))
    torch.cuda.synchronize()                             # the call's stream may start on these
    return s


def _records(out):
    f = out.view(torch.float32)
    return {"token": out[:, 0], "flags": out[:, 1], "stats": f[:, 2:]}      # entropy (nats, normalised), largest logit, ln sum exp


def run(s):
    c = s.c
    if c["kind"] == "route":
        P.rs_route(s.logits, c["n"], c["vocab"], s.scale, TAU, P.RS_SLM, s.out, s.scratch)
        return _records(s.out)
    if c["kind"] == "router_plus":
        P.binding.rs_route_plus(None, s.hidden, c["n"], s.router, P.RS_SLM, s.out, s.logits)
        return {"flags": s.out[:, 1], "logits": s.logits}
    if c["rows"] == c["seqs"]:
        P.rs_decode_step(s.m.handle, c["seqs"], s.slot, s.tok, s.pos, s.scale, TAU, s.active, s.out, s.logits, s.stream)
    else:
        P.rs_catchup_prefill(s.m.handle, c["seqs"], c["rows"], s.slot, s.tok, s.off, s.pos, s.scale, TAU, s.active, s.out,
                             s.logits, s.stream)
    torch.cuda.current_stream().wait_stream(s.stream)    # what follows on the caller's stream sees the results
    return {"record": _records(s.out), "logits": s.logits, "k": s.k, "v": s.v}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    if c["kind"] == "route":
        return {"bytes": 4 * c["n"] * c["vocab"] + 28 * c["n"], "flops": 4 * c["n"] * c["vocab"]}
    if c["kind"] == "router_plus":
        d, r = c["d"], c["r"]
        weights = 6 * (2 * r * d + r + d) + 4 * d + 2
        return {"bytes": 2 * weights + c["n"] * (4 * d + 8 + 8), "flops": 2 * c["n"] * weights}
    _, d, nq, nkv, hd, ffn, _ = SHAPES[c["shape"]]
    n_l, n, rows, V = c["layers"], c["seqs"], c["rows"], c["vocab"]
    span, ctx = _spans(c)
    per_layer = (nq + 2 * nkv) * hd * d + nq * hd * d + 3 * d * ffn
    kv_row = 2 * nkv * hd * 2                            # K and V of one position in one layer, bytes
    reads = n_l * (2 * per_layer + 4 * d) + 2 * V * d + 2 * d + 2 * rows * d + n_l * kv_row * sum(ctx)
    writes = n_l * kv_row * rows + 4 * n * V + 24 * n
    pairs = sum(x * s + s * (s + 1) // 2 for s, x in zip(span, ctx))       # (row, position it attends to)
    return {"bytes": reads + writes, "flops": n_l * (2 * per_layer * rows + 4 * nq * hd * pairs) + 2 * V * d * n}


def tolerance(case):
    c = case
    if c["kind"] == "route":
        # fp32 sums of up to 2e5 exponentials in another order
        return {"rel": 2e-6, "max": 2e-5}
    if c["kind"] == "router_plus":
        return {"rel": 1e-5, "max": 1e-4}
    # fp32 sums in another order; the K/V rows of the call are rounded to bf16, where a sum in another order now and
    # then rounds the other way (one step, 2^-8 of the value): the "max" of the caches, and a little of what the later rows
    # and layers of a span read.  Against 64 bits with that rounding: up to 5e-6 in the logits of decode steps, 1.3e-4 in
    # those of spans.
    return {"rel": 2e-5 if c["rows"] == c["seqs"] else 5e-4, "max": 2e-2, "differ": 0.01}


# ------------------------------------------------------------------ 64-bit values
def exact(case, seed):
    c = case
    if c["kind"] == "route":
        g = _gen(seed)
        x = _normal(g, (c["n"], c["vocab"]), 1.2, dtype=torch.float32).double()
        x *= torch.empty(c["n"], device="cuda").uniform_(0.5, 8.0, generator=g).double()[:, None]
        return dict(_exact_records(x), token=None, flags=None)
    if c["kind"] == "router_plus":
        x, w = _router_inputs(c, seed)
        x = x.double()
        for w1, b1, w2, b2 in zip(w.w1, w.b1, w.w2, w.b2):
            z = x @ w1.double().T + b1.double()
            x = x + (0.5 * z * (1 + torch.erf(z / math.sqrt(2)))) @ w2.double().T + b2.double()
        mu = x.mean(1, keepdim=True)
        y = (x - mu) / torch.sqrt(((x - mu) ** 2).mean(1, keepdim=True) + 1e-5) * w.ln_gain.double() + w.ln_bias.double()
        return {"flags": None, "logits": y @ w.w_head.double().T + w.b_head.double()}
    return _exact_call(c, seed)


def _exact_records(x):
    lse = torch.logsumexp(x, 1)
    h = lse - (torch.exp(x - lse[:, None]) * x).sum(1)
    return {"stats": torch.stack([h, h / math.log(x.shape[1]), x.max(1).values, lse], 1)}


def _exact_call(c, seed):
    """The decoder in fp64.  The caches that are returned hold the call's K/V rows before their rounding to bf16.  In a
    decode step attention reads the rounded row, as the cache holds it.  In a span it reads the rows of the call unrounded:
    which way a value near a rounding boundary falls depends on the last bit of its sum, and a later row of the same call
    reads it, so with rounding the distance to this function would be a matter of luck (2e-6 .. 2e-5 for one kernel on
    two seeds); without, it is that of the rounding itself, the same for every order of summation."""
    _, d, nq, nkv, hd, ffn, _ = SHAPES[c["shape"]]
    w, k, v, tok, scale = _call_inputs(c, seed)
    grp, half = nq // nkv, hd // 2
    span, ctx = _spans(c)
    slots = _slots(c["seqs"])
    kx, vx = k.double(), v.double()
    pos = torch.cat([torch.arange(x, x + s, device="cuda") for s, x in zip(span, ctx)]).double()
    ang = pos[:, None] * THETA ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / hd)
    cs, sn = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

    def norm(x, gain):
        return x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS) * gain.double()

    def rope(x):
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cs - b * sn, b * cs + a * sn], -1)

    h = w.embed[tok.long()].double()
    for l, lw in enumerate(w.layers):
        qkv = norm(h, lw.attn_norm) @ lw.w_qkv.double().T
        q = rope(qkv[:, :nq * hd].reshape(-1, nq, hd))
        kn = rope(qkv[:, nq * hd:(nq + nkv) * hd].reshape(-1, nkv, hd))
        vn = qkv[:, (nq + nkv) * hd:].reshape(-1, nkv, hd)
        o = torch.empty(c["rows"], nq, hd, dtype=torch.float64, device="cuda")
        r = 0
        for b, (s, x) in enumerate(zip(span, ctx)):
            sl = slots[b]
            k64, v64 = kn[r:r + s].transpose(0, 1), vn[r:r + s].permute(1, 2, 0)
            kx[l, sl, :, x:x + s], vx[l, sl, :, :, x:x + s] = k64, v64
            keys, vals = kx[l, sl, :, :x + s], vx[l, sl, :, :, :x + s]
            if c["rows"] == c["seqs"]:
                keys = torch.cat([keys[:, :x], k64.float().bfloat16().double()], 1)
                vals = torch.cat([vals[:, :, :x], v64.float().bfloat16().double()], 2)
            qb = q[r:r + s].reshape(s, nkv, grp, hd).permute(1, 0, 2, 3).reshape(nkv, s * grp, hd).contiguous()
            sc = torch.matmul(qb, keys.transpose(1, 2).contiguous()) / math.sqrt(hd)
            last = torch.arange(x, x + s, device="cuda").repeat_interleave(grp)
            sc = sc.masked_fill(torch.arange(x + s, device="cuda")[None] > last[:, None], -math.inf)
            ob = torch.matmul(torch.softmax(sc, 2), vals.transpose(1, 2).contiguous())
            o[r:r + s] = ob.reshape(nkv, s, grp, hd).permute(1, 0, 2, 3).reshape(s, nq, hd)
            r += s
        h = h + o.reshape(-1, nq * hd) @ lw.w_o.double().T
        gu = norm(h, lw.mlp_norm) @ lw.w_gate_up.double().T
        h = h + (torch.nn.functional.silu(gu[:, :ffn]) * gu[:, ffn:]) @ lw.w_down.double().T
    last = torch.tensor(span, device="cuda").cumsum(0) - 1
    x = norm(h[last], w.final_norm) @ w.lm_head.double().T * scale.double()[:, None]
    return {"record": dict(_exact_records(x), token=None, flags=None), "logits": x, "k": kx, "v": vx}


def _router_inputs(c, seed):
    """Hidden states of the magnitude a residual stream has, and a router as the package's workloads draw one."""
    g = _gen(seed)
    n, d, r = c["n"], c["d"], c["r"]
    hidden = _normal(g, (n, d), 1.0, dtype=torch.float32)
    w = SimpleNamespace(w1=[_normal(g, (r, d), 0.05) for _ in range(6)], b1=[_normal(g, (r,), 0.002) for _ in range(6)],
                        w2=[_normal(g, (d, r), 0.05) for _ in range(6)], b2=[_normal(g, (d,), 0.002) for _ in range(6)],
                        ln_gain=_normal(g, (d,), 0.1, 1.0), ln_bias=_normal(g, (d,), 0.1), w_head=_normal(g, (2, d), 0.05),
                        b_head=_normal(g, (2,), 0.05))
    return hidden, w
