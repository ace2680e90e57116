"""The calls whose speed this library answers for, from the smallest to the largest.

Each case is one pass through the public entry points (``attn``, ``ffn``, ``attn_dense``
and the autograd layers) at a size a program would use: the benchmark workloads
(``paper_2106_06899_amd.workloads``), the attention and feed-forward layers of the paper's
benchmarks, training steps, few queries against many keys, and odd sizes in both types.

Inputs are drawn on the GPU from the seed alone, by the recipes of the benchmark
workloads: N(0, 1) queries, keys and values; feed-forward weights N(0, 0.02^2); and, where
a case says ``planted``, queries that are the sum of four of their valid keys plus noise
(heads that look for something). In 32 bits that sum is doubled, so that the weight of the
k-th key is small and a tie at rank k that another order of summation breaks the other way
does not show in the result.
"""
from __future__ import annotations

import math

import torch

import paper_2106_06899_amd as tk
from paper_2106_06899_amd import layers

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _attn(name, op="attn", **kw):
    c = dict(op=op, dtype="bf16", B=1, H=1, Lq=0, Lk=0, d=64, k=64, chunk=1024, causal=False, planted=False)
    c.update(kw)
    return dict(c, name=name) if name else c


def _ffn(name, op="ffn", **kw):
    c = dict(op=op, dtype="bf16", N=0, d_model=768, d_ff=4096, k=512, chunk=1024)
    c.update(kw)
    return dict(c, name=name) if name else c


def _mha(name, **kw):
    c = dict(op="mha_train", dtype="bf16", B=1, L=1024, d_model=768, H=12, k=64, chunk=1024, causal=False)
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest benchmark workload: one 32-bit head, where launches and latency count
        _attn("attn_f32_one_head", dtype="f32", Lq=1024, Lk=1024, k=32, chunk=256, planted=True),
        # a BERT-base encoder layer's attention over a batch of 512-token sequences
        _attn("attn_encoder", B=8, H=12, Lq=512, Lk=512, chunk=512),
        # the long-sequence benchmark workload
        _attn("attn_long", H=16, Lq=32768, Lk=32768, planted=True),
        # a causal decoder's prefill over a batch of 8192-token sequences
        _attn("attn_causal_d128", B=4, H=16, Lq=8192, Lk=8192, d=128, k=128, causal=True),
        # a few new queries of a batch against long key sequences
        _attn("attn_few_queries", B=4, H=16, Lq=5, Lk=20001, d=128, k=128),
        # attention of the paper's causal layer benchmark, forward and backward
        _attn("attn_train_causal", op="attn_train", H=12, Lq=4096, Lk=4096, k=128, causal=True),
        # 32-bit training at odd sizes
        _attn("attn_train_f32_ragged", op="attn_train", dtype="f32", B=2, H=4, Lq=1511, Lk=1511, d=96, k=100,
              chunk=500, causal=True, planted=True),
        # query chunking with the top-k off, the comparison of the paper's layer benchmark
        _attn("attn_dense", op="dense", H=12, Lq=8192, Lk=8192, k=8192),
        # the feed-forward benchmark workload
        _ffn("ffn_wide", N=16384, d_model=1024, d_ff=65536),
        # feed-forward layer on a handful of tokens
        _ffn("ffn_few_tokens", N=24, d_model=768, d_ff=16384, k=256),
        # training step of the paper's feed-forward layer, on 32 sequences of 512 tokens
        _ffn("ffn_train", op="ffn_train", N=16384, d_ff=4096),
        # training step of a whole BERT-base attention layer, projections included
        _mha("mha_layer_train", B=4, L=1024),
    ]


# ----------------------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: the same kinds of call, sizes spread over their
    logarithm, most of them odd; costs are bounded by the largest listed case."""
    kind = rng.choice(["self", "self", "f32", "few_queries", "attn_train", "dense", "ffn", "ffn_few", "ffn_train", "mha"])
    chunk = rng.choice([0, 256, 512, 1024, 1000])
    if kind in ("self", "f32", "attn_train"):
        f32 = kind == "f32" or (kind == "attn_train" and rng.random() < 0.3)
        d = rng.choice([64, 64, 128, 128, 32, 96])
        heads = rng.choice([1, 2, 4, 8, 12, 16, 32, 64, 96])
        top = min(32768 if kind == "self" else 8192, int(math.sqrt((2e11 if f32 else 1.5e12) / (2.0 * d * heads))))
        L = _log(rng, 130, max(top, 200))
        k = max(1, min(_log(rng, 8, 256), L // 2))
        H = math.gcd(heads, 16) if heads % 12 else 12
        return _attn(None, op="attn_train" if kind == "attn_train" else "attn", dtype="f32" if f32 else "bf16",
                     B=heads // H, H=H, Lq=L, Lk=L, d=d, k=k, chunk=chunk, causal=rng.random() < 0.5,
                     planted=f32 or rng.random() < 0.5)
    if kind == "few_queries":
        d = rng.choice([64, 128])
        B, H = rng.choice([1, 2, 4, 8]), rng.choice([8, 12, 16])
        Lk = _log(rng, 1100, min(65000, int(2e9 / (4.0 * B * H * d))))
        return _attn(None, B=B, H=H, Lq=_log(rng, 1, 64), Lk=Lk, d=d, k=_log(rng, 8, 128), chunk=chunk)
    if kind == "dense":
        d, H = rng.choice([64, 128]), rng.choice([4, 12, 16])
        L = _log(rng, 300, int(math.sqrt(8e11 / (4.0 * d * H))))
        return _attn(None, op="dense", H=H, Lq=L, Lk=L, d=d, k=L, chunk=chunk, causal=rng.random() < 0.5)
    if kind in ("ffn", "ffn_few", "ffn_train"):
        dm = rng.choice([256, 512, 768, 1024])
        dff = _log(rng, 2048, 32768 if kind == "ffn_train" else 65536) // 8 * 8
        N = _log(rng, 1, 200) if kind == "ffn_few" else _log(rng, 500, 16384)
        k = max(1, min(_log(rng, 32, 512), dff // 4))
        return _ffn(None, op="ffn_train" if kind == "ffn_train" else "ffn", N=N, d_model=dm, d_ff=dff, k=k, chunk=chunk)
    dm, H = rng.choice([(512, 8), (768, 12), (1024, 16), (1024, 8)])
    L = _log(rng, 100, 3000)
    return _mha(None, B=max(1, min(8, 8192 // L)), L=L, d_model=dm, H=H, k=max(1, min(_log(rng, 16, 128), L // 2)),
                chunk=chunk, causal=rng.random() < 0.5)


# ----------------------------------------------------------------------------- inputs
def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = DTYPES[case["dtype"]]

    def normal(*shape, std=1.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(dt)

    s = {"case": case}
    if case["op"] in ("ffn", "ffn_train"):
        s["x"] = normal(case["N"], case["d_model"])
        s["w1"] = normal(case["d_ff"], case["d_model"], std=0.02)
        s["w2"] = normal(case["d_ff"], case["d_model"], std=0.02)
        if case["op"] == "ffn_train":
            s["g"] = normal(case["N"], case["d_model"])
            for n in ("x", "w1", "w2"):
                s[n].requires_grad_()
        return s
    if case["op"] == "mha_train":
        m = layers.TopkMultiheadAttention(case["d_model"], case["H"], case["k"], case["chunk"], case["causal"],
                                          device="cuda", dtype=dt)
        with torch.no_grad():  # torch.nn.Linear's own ranges, drawn from the seed
            for p in m.parameters():
                b = 1.0 / math.sqrt(case["d_model"])
                p.copy_((torch.rand(p.shape, generator=gen, device="cuda") * 2 - 1) * b)
        s["m"] = m
        s["x"] = normal(case["B"], case["L"], case["d_model"]).requires_grad_()
        s["g"] = normal(case["B"], case["L"], case["d_model"])
        return s
    B, H, Lq, Lk, d = (case[n] for n in ("B", "H", "Lq", "Lk", "d"))
    s["k"], s["v"] = normal(B, H, Lk, d), normal(B, H, Lk, d)
    if case["planted"]:
        i = torch.arange(Lq, device="cuda")
        valid = torch.clamp(i + 1, max=Lk) if case["causal"] else torch.full_like(i, Lk)
        acc = 0.5 * torch.randn(B, H, Lq, d, generator=gen, device="cuda")
        for _ in range(4):
            j = (torch.rand(B, H, Lq, generator=gen, device="cuda") * valid).long().clamp_(max=Lk - 1)
            acc += (2.0 if case["dtype"] == "f32" else 1.0) * torch.gather(s["k"].float(), 2, j[..., None].expand(-1, -1, -1, d))
        s["q"] = acc.to(dt)
    else:
        s["q"] = normal(B, H, Lq, d)
    if case["op"] == "attn_train":
        s["g"] = normal(B, H, Lq, d)
        for n in ("q", "k", "v"):
            s[n].requires_grad_()
    return s


# ----------------------------------------------------------------------------- one pass
def run(state):
    c = state["case"]
    op = c["op"]
    if op == "attn":
        return tk.attn(state["q"], state["k"], state["v"], c["k"], c["chunk"], c["causal"])
    if op == "dense":
        return tk.attn_dense(state["q"], state["k"], state["v"], c["chunk"], c["causal"])
    if op == "ffn":
        return tk.ffn(state["x"], state["w1"], state["w2"], c["k"], c["chunk"])
    if op == "attn_train":
        out = layers.topk_attention(state["q"], state["k"], state["v"], c["k"], c["chunk"], c["causal"])
        return (out.detach(),) + torch.autograd.grad(out, (state["q"], state["k"], state["v"]), state["g"])
    if op == "ffn_train":
        out = layers.topk_feed_forward(state["x"], state["w1"], state["w2"], c["k"], c["chunk"])
        return (out.detach(),) + torch.autograd.grad(out, (state["x"], state["w1"], state["w2"]), state["g"])
    out = state["m"](state["x"])
    return (out.detach(),) + torch.autograd.grad(out, (state["x"],) + tuple(state["m"].parameters()), state["g"])


# ----------------------------------------------------------------------------- compulsory work
def _pairs(case):
    """(valid (query, key) pairs, selected pairs) over every row of the call."""
    heads, Lq, Lk = case["B"] * case["H"], case.get("Lq") or case["L"], case.get("Lk") or case["L"]
    if not case["causal"]:
        return heads * Lq * Lk, heads * Lq * min(case["k"], Lk)

    def tri(cap):  # sum over i < Lq of min(i + 1, cap)
        n = min(Lq, cap)
        return n * (n + 1) // 2 + (Lq - n) * cap

    return heads * tri(Lk), heads * tri(min(case["k"], Lk))


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    op, d = case["op"], case.get("d") or case["d_model"]
    if op in ("ffn", "ffn_train"):
        rows, keys = case["N"], case["d_ff"]
        pairs, sel = rows * keys, rows * case["k"]
    elif op == "mha_train":
        d = case["d_model"] // case["H"]
        pairs, sel = _pairs(case)
        rows, D = case["B"] * case["L"], case["d_model"]
        # x, d_out in, out, d_x written; both weight matrices in, their gradients out
        return {"bytes": e * (4 * rows * D + 2 * (4 * D * D + 4 * D)),
                "flops": 2 * d * pairs + 10 * d * sel + 3 * 2 * rows * 4 * D * D}
    else:
        heads = case["B"] * case["H"]
        rows, keys = heads * case["Lq"], heads * case["Lk"]
        pairs, sel = _pairs(case)
    if op == "dense":
        return {"bytes": e * d * (2 * rows + 2 * keys), "flops": 4 * d * pairs}
    if op in ("attn", "ffn"):
        return {"bytes": e * d * (2 * rows + 2 * keys), "flops": 2 * d * pairs + 2 * d * sel}
    # forward and backward: queries, output gradient, keys and values in; output and the
    # three gradients out; four more products per selected pair
    return {"bytes": e * d * (4 * rows + 4 * keys), "flops": 2 * d * pairs + 10 * d * sel}


# ----------------------------------------------------------------------------- what the result is
def tolerance(case):
    """32 bits: sums of up to a few thousand terms in another order. bf16: the rounding of
    the stored result (2^-9 per element at most, 1.7e-3 in the 2-norm), four times."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 7e-3}


def _exact_heads(q, k, v, topk, scale, causal, relu, g=None):
    """Top-k attention of one head (or the feed-forward layer) in 64 bits, 512 rows at a
    time: the selected weights are scattered into a dense row and multiplied."""
    q, k, v = q.double(), k.double(), v.double()
    Lq, Lk = q.shape[0], k.shape[0]
    kt, vt = k.t().contiguous(), v.t().contiguous()
    out = torch.empty_like(q)
    dq = torch.empty_like(q)
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    for r0 in range(0, Lq, 512):
        qi = q[r0:r0 + 512]
        s = qi @ kt
        if causal:
            i = torch.arange(r0, r0 + qi.shape[0], device=q.device)
            s.masked_fill_(torch.arange(Lk, device=q.device)[None] > i[:, None], -math.inf)
        top, idx = torch.topk(s, topk, dim=1)
        w = torch.relu(top) if relu else torch.softmax(top * scale, dim=1)
        P = torch.zeros_like(s).scatter_(1, idx, w)
        out[r0:r0 + 512] = P @ v
        if g is None:
            continue
        gi = g[r0:r0 + 512].double()
        a = torch.gather(gi @ vt, 1, idx)
        ds = a * (top > 0) if relu else scale * w * (a - (w * a).sum(1, keepdim=True))
        D = torch.zeros_like(s).scatter_(1, idx, ds)
        dq[r0:r0 + 512] = D @ k
        dk += D.t().contiguous() @ qi
        dv += P.t().contiguous() @ gi
    return out if g is None else (out, dq, dk, dv)


def exact(case, seed):
    op = case["op"]
    if op == "mha_train":  # its selection follows the projections' 16-bit rounding
        return None
    s = prepare(case, seed)
    with torch.no_grad():
        if op in ("ffn", "ffn_train"):
            return _exact_heads(s["x"], s["w1"], s["w2"], case["k"], 1.0, False, True, s.get("g"))
        scale = 1.0 / math.sqrt(case["d"])
        outs = []
        for b in range(case["B"]):
            for h in range(case["H"]):
                q, k, v = (s[n][b, h] for n in ("q", "k", "v"))
                g = s["g"][b, h] if "g" in s else None
                if op == "dense":
                    o = torch.empty(q.shape, dtype=torch.float64, device=q.device)
                    kt, vd = k.double().t().contiguous(), v.double()
                    for r0 in range(0, q.shape[0], 512):
                        t = (q[r0:r0 + 512].double() @ kt) * scale
                        if case["causal"]:
                            i = torch.arange(r0, r0 + t.shape[0], device=q.device)
                            t.masked_fill_(torch.arange(k.shape[0], device=q.device)[None] > i[:, None], -math.inf)
                        o[r0:r0 + 512] = torch.softmax(t, dim=1) @ vd
                    outs.append(o)
                else:
                    outs.append(_exact_heads(q, k, v, case["k"], scale, case["causal"], False, g))
        shape = (case["B"], case["H"])
        if isinstance(outs[0], tuple):
            return tuple(torch.stack([o[t] for o in outs]).view(*shape, *outs[0][t].shape) for t in range(4))
        return torch.stack(outs).view(*shape, *outs[0].shape)
