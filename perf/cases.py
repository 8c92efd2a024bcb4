"""Performance cases of the masked projections, attention and router.

Every case is one pass through the public entry points of
``paper_2607_28418_amd``, with the buffers a serving program keeps (weights,
caches, workspaces, outputs) made once in ``prepare``.  The families are the
operators of a width-pruned decoder layer:

  ffn          masked SwiGLU FFN: decode batches, prompts, long prefills;
               groups from 16 channels up, bf16 and fp32
  proj         the attention projections under one routing decision: the mask
               reorder (prefill only), masked Q with dense K and V, masked O
  attn         masked prefill attention: causal or full, several sequences,
               cached prefixes (T_k > T_q) and left padding
  attn_decode  masked decode attention over ragged caches, both layouts
  router       bottleneck router, with the logits and the reorder of its mask

Inputs follow the distributions of the workloads in ``synth.py``: activations
N(0, 1), weights N(0, 0.02^2), masks from the top-k of a random projection of
the tokens, from per-group Beta(2,2) probabilities, or Bernoulli.
"""
import math

import torch

import paper_2607_28418_amd as W

DECODE_MAX = 64     # tokens up to which a bf16 call is a decode call: it needs no reorder
HEAD_DIM = 128


# ---- the cases ---------------------------------------------------------------------

def listed():
    ffn7b = dict(op="ffn", dtype="bf16", d_model=4096, d_ff=11008, group=128, keep=0.5)
    ffn8b = dict(op="ffn", dtype="bf16", d_model=4096, d_ff=14336, group=128, keep=0.5)
    gqa = dict(op="proj", d_model=4096, n_q=32, n_kv=8, group=512, keep=0.5, mask="topk")
    heads = dict(n_q=32, n_kv=8, group=512, keep=0.5)
    return [
        # one user generating: every token is one such call per layer (Llama-7B widths)
        dict(ffn7b, name="ffn_decode_b1", M=1, mask="beta"),
        # a serving batch generating together (Llama-3-8B widths)
        dict(ffn8b, name="ffn_decode_b32", M=32, mask="topk"),
        # a chat prompt of ordinary, odd length, or a chunk of a chunked prefill
        dict(ffn8b, name="ffn_prompt_t300", M=300, mask="topk"),
        # a long document, the widths and length the layer benchmark uses
        dict(ffn8b, name="ffn_prefill_t8192", M=8192, mask="topk"),
        # fine-grained routing: 32-channel groups on a ragged prompt
        dict(ffn7b, name="ffn_narrow_groups_t2000", M=2000, group=32, mask="topk"),
        # the fp32 configuration (reference numerics of a small model)
        dict(op="ffn", name="ffn_fp32_t128", dtype="f32", M=128, d_model=512, d_ff=1536, group=64, keep=0.5,
             mask="bernoulli"),
        # attention projections of a mid-size prompt, multi-head (no GQA), odd length
        dict(gqa, name="proj_mha_t777", M=777, n_kv=32),
        # attention projections of a long prefill, grouped queries
        dict(gqa, name="proj_gqa_t8192", M=8192),
        # causal attention of the long prefill
        dict(heads, op="attn", name="attn_t8192", n_seq=1, T_q=8192, T_k=8192, causal=True, leftpad=False),
        # a batch of prompt chunks against cached prefixes
        dict(heads, op="attn", name="attn_chunks_4x500", n_seq=4, T_q=500, T_k=1500, causal=True, leftpad=False),
        # decode attention of a serving batch, sequences of different ages
        dict(heads, op="attn_decode", name="attn_decode_b32", B=32, L=8192, ragged=True, head_major=False,
             mask="bernoulli"),
        # routing decision of the FFN for the long prefill
        dict(op="router", name="router_t8192", M=8192, d_model=4096, rank=16, groups=112),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["ffn", "ffn", "ffn", "ffn", "ffn32", "proj", "proj", "attn", "attn", "attn_decode", "router"])
    keep = rng.choice([0.25, 0.5, 0.5, 0.75])
    if op == "ffn":
        d_model, d_ff = rng.choice([(4096, 11008), (4096, 14336), (4096, 14336), (2048, 8192), (1024, 4096)])
        M = _log_int(rng, 1, 8192 if keep <= 0.5 else 4096)
        mask = rng.choice(["topk", "bernoulli"] + (["beta"] if keep == 0.5 else []))
        # groups below 64 channels compute every block, so they are drawn up to half the length
        group = rng.choice([128, 128, 128, 64, 256, 32, 16])
        if group < 64:
            M = min(M, 4096)
        return dict(op="ffn", dtype="bf16", M=M, d_model=d_model, d_ff=d_ff, group=group, keep=keep, mask=mask)
    if op == "ffn32":
        group = rng.choice([16, 32, 64, 128])
        return dict(op="ffn", dtype="f32", M=_log_int(rng, 1, 512), d_model=rng.choice([256, 512, 768, 1024]),
                    d_ff=group * rng.randint(256 // group, 2048 // group), group=group, keep=keep, mask="bernoulli")
    n_q, n_kv, group = rng.choice([(32, 8, 512), (32, 8, 512), (32, 32, 512), (32, 8, 128), (32, 8, 1024),
                                   (16, 4, 256), (16, 16, 256)])
    heads = dict(n_q=n_q, n_kv=n_kv, group=group, keep=keep)
    if op == "proj":
        return dict(heads, op="proj", M=_log_int(rng, 1, 8192), d_model=n_q * HEAD_DIM,
                    mask=rng.choice(["topk", "bernoulli"]))
    if op == "attn":
        n_seq = rng.choice([1, 1, 1, 2, 3, 4, 8])
        T_q = _log_int(rng, 32, 8192 // n_seq)
        T_k = T_q + rng.choice([0, 0, rng.randint(1, max(1, 8192 // n_seq - T_q + 1))])
        causal = rng.random() < 0.8
        if not causal:
            T_q, T_k = min(T_q, 2048), min(T_k, 4096)
        return dict(heads, op="attn", n_seq=n_seq, T_q=T_q, T_k=T_k, causal=causal, leftpad=rng.random() < 0.25)
    if op == "attn_decode":
        B = _log_int(rng, 1, 64)
        return dict(heads, op="attn_decode", B=B, L=_log_int(rng, 64, min(8192, 262144 // B)),
                    ragged=rng.random() < 0.7, head_major=rng.random() < 0.4,
                    mask=rng.choice(["bernoulli", "topk"]))
    return dict(op="router", M=_log_int(rng, 1, 8192), d_model=rng.choice([2048, 4096, 4096]),
                rank=rng.choice([8, 16, 32]), groups=rng.choice([8, 32, 86, 112]))


# ---- inputs ------------------------------------------------------------------------

def _mask(g, kind, x, n_groups, keep):
    """uint8 [tokens][n_groups] drawn as the workloads' masks are."""
    M = x.shape[0]
    if kind == "topk":  # round half up, as the routers' keep count
        k = int(math.floor(n_groups * keep + 0.5))
        R = torch.randn(x.shape[1], n_groups, generator=g, device="cuda")
        top = (x.float() @ R).topk(k, dim=1).indices
        return torch.zeros(M, n_groups, dtype=torch.uint8, device="cuda").scatter_(1, top, 1)
    p = keep
    if kind == "beta":  # Beta(2,2): the middle one of three uniform draws
        p = torch.rand(3, n_groups, generator=g, device="cuda").median(dim=0).values
        p = (p * (keep / p.mean())).clamp(0.0, 1.0)
    return (torch.rand(M, n_groups, generator=g, device="cuda") < p).to(torch.uint8)


def _inputs(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = torch.float32 if c.get("dtype") == "f32" else torch.bfloat16

    def normal(*shape, std=1.0):
        return (torch.randn(*shape, generator=g, device="cuda") * std).to(dt)

    if c["op"] == "ffn":
        D, F = c["d_model"], c["d_ff"]
        x = normal(c["M"], D)
        return dict(x=x, w_gate=normal(F, D, std=0.02), w_up=normal(F, D, std=0.02), w_down=normal(D, F, std=0.02),
                    mask=_mask(g, c["mask"], x, F // c["group"], c["keep"]))
    if c["op"] == "router":
        D, r = c["d_model"], c["rank"]
        return dict(x=normal(c["M"], D), w1=normal(r, D, std=0.02), w2=normal(2 * c["groups"], r, std=0.3))
    nq, nkv = c["n_q"] * HEAD_DIM, c["n_kv"] * HEAD_DIM
    ng = nq // c["group"]
    if c["op"] == "proj":
        D = c["d_model"]
        x = normal(c["M"], D)
        return dict(x=x, a=normal(c["M"], nq), w_q=normal(nq, D, std=0.02), w_k=normal(nkv, D, std=0.02),
                    w_v=normal(nkv, D, std=0.02), w_o=normal(D, nq, std=0.02),
                    mask=_mask(g, c["mask"], x, ng, c["keep"]))
    if c["op"] == "attn":
        n, T_q, T_k = c["n_seq"], c["T_q"], c["T_k"]
        q = normal(n * T_q, nq)
        pad = None
        if c["leftpad"]:  # prompts of different lengths, batched with padding in front
            pad = torch.randint(0, T_k // 2 + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
        return dict(q=q, k=normal(n * T_k, nkv), v=normal(n * T_k, nkv), leftpad=pad,
                    mask=_mask(g, "topk", q, ng, c["keep"]))
    B, L = c["B"], c["L"]
    shape = (B, c["n_kv"], L, HEAD_DIM) if c["head_major"] else (B, L, nkv)
    q = normal(B, nq)
    kv_len = None
    if c["ragged"]:
        kv_len = torch.randint(1, L + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    return dict(q=q, k=normal(*shape), v=normal(*shape), kv_len=kv_len, mask=_mask(g, c["mask"], q, ng, c["keep"]))


def _ws(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def prepare(c, seed):
    """Inputs and weights, with the output and workspace buffers that a serving program keeps."""
    s = dict(_inputs(c, seed), case=c)
    if c["op"] == "ffn":
        dt = W.F32 if c["dtype"] == "f32" else W.BF16
        s["y"] = torch.empty_like(s["x"])
        s["ws"] = _ws(W.wide_workspace_size(W.OP_FFN, dt, c["M"], c["d_model"], c["d_ff"], c["group"]))
    elif c["op"] == "proj":
        M, D, nq, nkv = c["M"], c["d_model"], c["n_q"] * HEAD_DIM, c["n_kv"] * HEAD_DIM
        ng = nq // c["group"]
        x = s["x"]
        s.update(q=x.new_empty(M, nq), k=x.new_empty(M, nkv), v=x.new_empty(M, nkv), y=x.new_empty(M, D),
                 idx=x.new_empty((ng, M), dtype=torch.int32), counts=x.new_empty((ng,), dtype=torch.int32))
        # the three calls follow each other on one stream and share the workspace
        s["ws"] = _ws(max(W.wide_workspace_size(W.OP_REORDER, W.BF16, M, 0, ng, 1),
                          W.wide_workspace_size(W.OP_QKV, W.BF16, M, D, nq, c["group"]),
                          W.wide_workspace_size(W.OP_O, W.BF16, M, D, nq, c["group"])))
    elif c["op"] == "attn":
        s["o"] = torch.empty_like(s["q"])
        s["ws"] = _ws(W.wide_attention_workspace_size(c["n_seq"], c["T_q"], c["T_k"], c["n_q"], c["n_kv"], HEAD_DIM,
                                                      c["group"], True))
    elif c["op"] == "attn_decode":
        s["o"] = torch.empty_like(s["q"])
        s["ws"] = _ws(W.wide_attention_decode_workspace_size(c["B"], c["L"], c["n_q"], c["n_kv"], HEAD_DIM,
                                                             c["group"]))
    else:
        M, ng = c["M"], c["groups"]
        x = s["x"]
        s.update(mask=x.new_empty((M, ng), dtype=torch.uint8), idx=x.new_empty((ng, M), dtype=torch.int32),
                 counts=x.new_empty((ng,), dtype=torch.int32))
        s["ws"] = _ws(W.wide_workspace_size(W.OP_ROUTER, W.BF16, M, c["d_model"], ng, c["rank"]))
    return s


def run(s):
    c = s["case"]
    if c["op"] == "ffn":
        return W.wide_ffn_masked(s["x"], s["w_gate"], s["w_up"], s["w_down"], s["mask"], c["group"], y=s["y"],
                                 ws=s["ws"])
    if c["op"] == "proj":
        heads = (c["group"], c["n_q"], c["n_kv"], HEAD_DIM)
        idx = counts = None
        if c["M"] > DECODE_MAX:
            idx, counts = W.wide_mask_reorder(s["mask"], idx=s["idx"], counts=s["counts"], ws=s["ws"])
        q, k, v = W.wide_qkvo_masked(W.PHASE_QKV, s["x"], s["mask"], *heads, w_q=s["w_q"], w_k=s["w_k"],
                                     w_v=s["w_v"], idx=idx, counts=counts, q=s["q"], k=s["k"], v=s["v"], ws=s["ws"])
        y = W.wide_qkvo_masked(W.PHASE_O, s["a"], s["mask"], *heads, w_o=s["w_o"], idx=idx, counts=counts, y=s["y"],
                               ws=s["ws"])
        return q, k, v, y
    if c["op"] == "attn":
        return W.wide_attention_masked(s["q"], s["k"], s["v"], s["mask"], c["n_seq"], c["n_q"], c["n_kv"], HEAD_DIM,
                                       c["group"], c["causal"], o=s["o"], ws=s["ws"], leftpad=s["leftpad"])
    if c["op"] == "attn_decode":
        return W.wide_attention_decode(s["q"], s["k"], s["v"], s["mask"], c["n_q"], c["n_kv"], HEAD_DIM, c["group"],
                                       kv_len=s["kv_len"], o=s["o"], ws=s["ws"], head_major=c["head_major"])
    return W.wide_router(s["x"], s["w1"], s["w2"], mask=s["mask"], logits=True, reorder=True, idx=s["idx"],
                         counts=s["counts"], ws=s["ws"])


# ---- what a pass cannot do without ---------------------------------------------------

def _union(c, tokens, n_groups):
    """Expected share of the groups that some token uses."""
    if c["mask"] == "beta":  # E[1 - (1 - p)^tokens] for p ~ Beta(2,2)
        return 1.0 - 6.0 / ((tokens + 2) * (tokens + 3))
    return 1.0 - (1.0 - c["keep"]) ** tokens


def _visible(c):
    """(query, key) pairs of one head and sequence, half the keys' average padding left out."""
    T_q, T_k = c["T_q"], c["T_k"]
    pairs = T_q * T_k - T_q * (T_q - 1) // 2 if c["causal"] else T_q * T_k
    if c["leftpad"]:
        pairs -= min(pairs // 2, T_q * (T_k // 4))
    return pairs


def work(c):
    if c["op"] == "ffn":
        M, D, F = c["M"], c["d_model"], c["d_ff"]
        e = 4 if c["dtype"] == "f32" else 2
        weights = 3 * D * F * _union(c, M, F // c["group"])
        return {"bytes": e * (weights + 2 * M * D) + M * F // c["group"], "flops": 6.0 * M * D * F * c["keep"]}
    if c["op"] == "router":
        M, D, r, ng = c["M"], c["d_model"], c["rank"], c["groups"]
        return {"bytes": 2 * (M * D + r * D + 2 * ng * r) + M * ng * (1 + 8 + 4) + 4 * ng,
                "flops": 2.0 * M * r * (D + 2 * ng)}
    nq, nkv, keep = c["n_q"] * HEAD_DIM, c["n_kv"] * HEAD_DIM, c["keep"]
    ng = nq // c["group"]
    if c["op"] == "proj":
        M, D = c["M"], c["d_model"]
        weights = 2 * D * nq * _union(c, M, ng) + 2 * D * nkv
        rows = 2 * M * D + M * nq * (1 + keep) + 2 * M * nkv
        order = 4 * (M * ng + ng) if M > DECODE_MAX else 0
        return {"bytes": 2 * (weights + rows) + M * ng + order, "flops": M * D * (4.0 * nq * keep + 4.0 * nkv)}
    if c["op"] == "attn":
        tokens, keys = c["n_seq"] * c["T_q"], c["n_seq"] * c["T_k"]
        return {"bytes": 2 * (tokens * nq * (1 + keep) + 2 * keys * nkv) + tokens * ng,
                "flops": 4.0 * HEAD_DIM * c["n_seq"] * _visible(c) * c["n_q"] * keep}
    keys = c["B"] * c["L"] * (0.5 if c["ragged"] else 1.0)
    per_kv = max(1, c["n_q"] // c["n_kv"] * HEAD_DIM // c["group"])  # groups that share one KV head
    used = 1.0 - (1.0 - keep) ** per_kv
    return {"bytes": 2 * (2 * keys * nkv * used + c["B"] * nq * (1 + keep)) + c["B"] * ng,
            "flops": 4.0 * HEAD_DIM * keys * c["n_q"] * keep}


# ---- reference in 64 bits -------------------------------------------------------------

def exact(c, seed):
    s = _inputs(c, seed)
    d = {k: v.double() for k, v in s.items() if v is not None and v.is_floating_point() and c["op"] != "attn_decode"}
    if c["op"] == "ffn":
        on = (s["mask"] != 0).repeat_interleave(c["group"], dim=1)
        h = torch.nn.functional.silu(d["x"] @ d["w_gate"].T) * (d["x"] @ d["w_up"].T) * on
        return h @ d["w_down"].T
    if c["op"] == "router":  # the mask and its reorder are whole numbers, decided by the logits
        return None, (d["x"] @ d["w1"].T) @ d["w2"].T, None, None
    on = (s["mask"] != 0).repeat_interleave(c["group"], dim=1)
    if c["op"] == "proj":
        return ((d["x"] @ d["w_q"].T) * on, d["x"] @ d["w_k"].T, d["x"] @ d["w_v"].T, (d["a"] * on) @ d["w_o"].T)
    per_kv = c["n_q"] // c["n_kv"]
    if c["op"] == "attn":
        n, T_q, T_k = c["n_seq"], c["T_q"], c["T_k"]
        q, k, v = (d[i].view(n, -1, h, HEAD_DIM) for i, h in (("q", c["n_q"]), ("k", c["n_kv"]), ("v", c["n_kv"])))
        o = torch.zeros_like(q)
        keys = torch.arange(T_k, device="cuda")[None, :]
        for b in range(n):
            seen = torch.ones(T_q, T_k, dtype=torch.bool, device="cuda")
            if c["causal"]:
                seen &= keys <= torch.arange(T_q, device="cuda")[:, None] + (T_k - T_q)
            if s["leftpad"] is not None:
                seen &= keys >= s["leftpad"][b]
            for h in range(c["n_q"]):
                sc = (q[b, :, h] @ k[b, :, h // per_kv].T) / math.sqrt(HEAD_DIM)
                p = torch.softmax(sc.masked_fill(~seen, float("-inf")), dim=1)
                o[b, :, h] = torch.nan_to_num(p) @ v[b, :, h // per_kv]  # (no visible key: zeros)
        return o.view(n * T_q, -1) * on
    q = s["q"].double().view(c["B"], c["n_kv"], per_kv, HEAD_DIM)
    o = torch.zeros_like(q)
    for b in range(c["B"]):
        n = c["L"] if s["kv_len"] is None else int(s["kv_len"][b])
        if c["head_major"]:
            k, v = s["k"][b, :, :n].double(), s["v"][b, :, :n].double()
        else:
            k, v = (s[i][b, :n].double().view(n, c["n_kv"], HEAD_DIM).transpose(0, 1).contiguous() for i in ("k", "v"))
        for h in range(c["n_kv"]):
            o[b, h] = torch.softmax((q[b, h] @ k[h].T) / math.sqrt(HEAD_DIM), dim=1) @ v[h]
    return o.view(c["B"], -1) * on


def tolerance(c):
    if c["op"] == "router":  # fp32 logits; a near tie may fall the other way and shift its column of the reorder
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.005}
    if c.get("dtype") == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}
