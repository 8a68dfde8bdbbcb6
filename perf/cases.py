"""The work whose speed is measured: calls of the public entry points over the sizes a user has.

Seven kinds of call, each at sizes of the models this repository serves (Mistral-7B:
32 query heads over 8 KV heads of 128; LLaMA-7B: 32 heads of 128; LLaMA-125M and GPT-2
small: 12 heads of 64), with keys a quarter of the head's width unless stated:

  decode    one decode step's attention over a cache (contiguous or paged; bf16, fp8
            or 4-bit keys; equal or ragged lengths)
  prefill   attention of a whole prompt, or of a chunk of it after a cached prefix
  train     attention forward with the log-sum-exp, then its backward
  project   the three projections of a layer converted to thin keys: of a prompt, or
            of one token per sequence
  append    a prompt's new rows written to the cache
  layer     a converted layer's whole decode step: three projections, the append and
            the decode

A serving loop runs the same decode step on the same buffers token after token, so the
one-token kinds call the prepared form that such a program keeps; prompts and training
steps differ from call to call and use the plain entry points.
"""
import math

import torch

import paper_2603_04427_amd as tk

# d_model, query heads, KV heads, head width
MODELS = {
    "mistral-7b": (4096, 32, 8, 128),
    "llama-7b": (4096, 32, 32, 128),
    "llama-125m": (768, 12, 12, 64),
    "gpt2": (768, 12, 12, 64),
}


def listed():
    return [
        # a single user's next token: the smallest call, where latency is what counts
        dict(name="decode_one_user", kind="decode", model="mistral-7b", r=32, batch=1, ctx=4096, keys="bf16",
             paged=False, block=0, ragged=False),
        # a small serving batch whose sequences have different lengths
        dict(name="decode_batch16_ragged", kind="decode", model="mistral-7b", r=32, batch=16, ctx=4096, keys="bf16",
             paged=False, block=0, ragged=True),
        # a large serving batch over long documents: fp8 keys in pages, the largest cache
        dict(name="decode_long_paged_fp8", kind="decode", model="mistral-7b", r=32, batch=32, ctx=32768, keys="fp8",
             paged=True, block=256, ragged=False),
        # a GPT-2-sized prompt in fp32, for callers that need fp32 accuracy
        dict(name="prefill_gpt2_f32", kind="prefill", model="gpt2", r=16, batch=1, seq_q=1024, seq_k=1024,
             dtype="f32", causal=True),
        # chunked prefill: the next 500 tokens of one long prompt against its cached prefix
        dict(name="prefill_chunk", kind="prefill", model="mistral-7b", r=32, batch=1, seq_q=500, seq_k=7700,
             dtype="bf16", causal=True),
        # the prompts of a batch, 8192 tokens each: the largest prefill
        dict(name="prefill_batch4_8k", kind="prefill", model="mistral-7b", r=32, batch=4, seq_q=8192, seq_k=8192,
             dtype="bf16", causal=True),
        # a training step's attention of a small from-scratch model, at an odd length
        dict(name="train_125m", kind="train", model="llama-125m", r=32, batch=8, seq=1000),
        # a training step's attention at 7B size with grouped queries
        dict(name="train_7b_gqa", kind="train", model="mistral-7b", r=32, batch=2, seq=4096),
        # the projections of a decode step: one token for each of 16 sequences
        dict(name="project_decode16", kind="project", model="mistral-7b", r=32, batch=16, seq=1),
        # the projections of a batch's prompts
        dict(name="project_prompts_8k", kind="project", model="mistral-7b", r=32, batch=4, seq=8192),
        # the prompts' rows written to a paged cache, keys quantised on the way in
        dict(name="append_prompts_fp8", kind="append", model="mistral-7b", r=32, batch=4, n_new=8192, ctx=8192,
             keys="fp8", paged=True, block=256),
        # a converted layer's whole decode step
        dict(name="layer_decode16", kind="layer", model="mistral-7b", r=32, batch=16, ctx=4096, keys="bf16",
             paged=True, block=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, model, least=16):
    """Key width: mostly a quarter of the head, sometimes half of it or all of it."""
    d = MODELS[model][3]
    return max(least, rng.choice([d // 4, d // 4, d // 4, d // 2, d]))


def _seconds(case):
    """A rough price of a case, to keep a drawn one below the largest listed one."""
    w = work(case)
    rate = 6e13 if case.get("dtype") == "f32" else 5e14 if case["kind"] == "train" else 1e15
    return max(w["bytes"] / 6e12, w["flops"] / rate) + 5e-6


def draw(rng):
    most = max(_seconds(c) for c in listed())
    cache = max(work(c)["bytes"] for c in listed())
    while True:
        kind = rng.choice(["decode", "decode", "prefill", "prefill", "train", "project", "project", "append", "layer"])
        model = rng.choice(list(MODELS))
        c = dict(kind=kind, model=model, r=_width(rng, model, 32 if kind == "train" else 16))
        if kind in ("decode", "append", "layer"):
            paged = rng.random() < 0.5
            c.update(batch=_log_int(rng, 1, 64), ctx=_log_int(rng, 100, 131072), paged=paged,
                     block=rng.choice([64, 128, 256]) if paged else 0,
                     keys=rng.choice(["bf16", "bf16", "fp8", "int4"]))
        if kind == "decode":
            c.update(ragged=rng.random() < 0.5)
        elif kind == "append":
            c.update(batch=_log_int(rng, 1, 16))
            c.update(n_new=_log_int(rng, 1, c["ctx"]))
        elif kind == "prefill":
            seq_q = _log_int(rng, 16, 8192)
            c.update(batch=_log_int(rng, 1, 8), seq_q=seq_q, seq_k=seq_q + rng.choice([0, _log_int(rng, 1, 16384)]),
                     dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), causal=rng.random() < 0.9)
        elif kind == "train":
            c.update(batch=_log_int(rng, 1, 16), seq=_log_int(rng, 64, 8192))
        elif kind == "project":
            one = rng.random() < 0.5
            c.update(batch=_log_int(rng, 1, 128) if one else _log_int(rng, 1, 8),
                     seq=1 if one else _log_int(rng, 2, 8192))
        if _seconds(c) <= most and _cache_bytes(c) <= cache:
            return c


def _cache_bytes(c):
    if "ctx" not in c:
        return 0
    _, _, h_kv, d = MODELS[c["model"]]
    return c["batch"] * h_kv * c["ctx"] * (_key_row(c) + 2 * d)


# ------------------------------------------------------------------ inputs


def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + salt)
    return g


def _randn(g, *shape, std=1.0, dtype=torch.bfloat16):
    """N(0, std^2) entries: activations behind a norm, and their projections."""
    x = torch.randn(*shape, generator=g, device="cuda", dtype=dtype)
    return x.mul_(std) if std != 1.0 else x


def _key_row(c):
    """Bytes of a cached key row with its scale."""
    return {"bf16": 2 * c["r"], "fp8": c["r"] + 4, "int4": c["r"] // 2 + 4}[c["keys"]]


def _quantise(k, keys):
    """Codes and scales of key rows, as the cache holds them: scale max|k| / 448 (E4M3) or / 7 (4-bit)."""
    k = k.float()
    amax = k.abs().amax(dim=-1)
    scale = torch.where(amax > 0, amax / (448.0 if keys == "fp8" else 7.0), torch.ones_like(amax))
    if keys == "fp8":
        return (k / scale[..., None]).to(torch.float8_e4m3fn).view(torch.uint8), scale
    n = torch.round(k / scale[..., None]).clamp_(-7, 7).to(torch.int8) + 8
    return (n[..., 0::2] | (n[..., 1::2] << 4)).to(torch.uint8), scale


def _dequantise(codes, scale, keys):
    """Key rows in 64 bits."""
    if keys == "bf16":
        return codes.double()
    if keys == "fp8":
        return codes.view(torch.float8_e4m3fn).double() * scale.double()[..., None]
    n = torch.stack([codes & 15, codes >> 4], dim=-1).flatten(-2)
    return (n.double() - 8) * scale.double()[..., None]


def _cache(c, seed, empty=False):
    """K, V, scales, block table of a cache of `ctx` positions a sequence."""
    _, _, h_kv, d = MODELS[c["model"]]
    g = _gen(seed, 1)
    table = None
    if c["paged"]:
        per = -(-c["ctx"] // c["block"])
        n = c["batch"] * per
        order = torch.randperm(n, generator=torch.Generator().manual_seed(seed + 17))
        table = order.view(c["batch"], per).to(torch.int32).cuda()
        lead = (n, h_kv, c["block"])
    else:
        lead = (c["batch"], h_kv, c["ctx"])
    width = c["r"] // 2 if c["keys"] == "int4" else c["r"]
    if empty:
        k = torch.zeros(*lead, width, dtype=torch.bfloat16 if c["keys"] == "bf16" else torch.uint8, device="cuda")
        return k, torch.zeros(*lead, d, dtype=torch.bfloat16, device="cuda"), \
            None if c["keys"] == "bf16" else torch.zeros(*lead, device="cuda"), table
    v = _randn(g, *lead, d)
    if c["keys"] == "bf16":
        return _randn(g, *lead, c["r"]), v, None, table
    k = torch.empty(*lead, width, dtype=torch.uint8, device="cuda")
    ks = torch.empty(*lead, device="cuda")
    for i in range(lead[0]):
        k[i], ks[i] = _quantise(_randn(g, *lead[1:], c["r"]), c["keys"])
    return k, v, ks, table


def _lens(c, seed):
    """Cached tokens of each sequence: all of `ctx`, or spread from an eighth of it to all of it."""
    if not c.get("ragged"):
        return torch.full((c["batch"],), c["ctx"], dtype=torch.int32, device="cuda")
    u = torch.rand(c["batch"], generator=torch.Generator().manual_seed(seed + 29))
    lens = (c["ctx"] * (0.125 + 0.875 * u)).to(torch.int32).clamp_(min=1)
    lens[0] = c["ctx"]
    return lens.cuda()


def _weights(c, seed):
    """Wt of q', k', v: logits q'.k' / sqrt(r) of standard deviation about 2."""
    d_model, h_q, h_kv, d = MODELS[c["model"]]
    g = _gen(seed, 2)
    s = 1.0 / math.sqrt(d_model)
    return (_randn(g, h_q * c["r"], d_model, std=2 * s), _randn(g, h_kv * c["r"], d_model, std=s),
            _randn(g, h_kv * d, d_model, std=s))


def _qkv(c, seed):
    _, h_q, h_kv, d = MODELS[c["model"]]
    g = _gen(seed, 3)
    dt = torch.float32 if c.get("dtype") == "f32" else torch.bfloat16
    sq = c["seq_q"] if "seq_q" in c else c["seq"]
    sk = c["seq_k"] if "seq_k" in c else c["seq"]
    return (_randn(g, c["batch"], h_q, sq, c["r"], std=2.0, dtype=dt), _randn(g, c["batch"], h_kv, sk, c["r"], dtype=dt),
            _randn(g, c["batch"], h_kv, sk, d, dtype=dt))


def prepare(case, seed):
    c = case
    d_model, h_q, h_kv, d = MODELS[c["model"]]
    st = {"case": c}
    if c["kind"] == "decode":
        k, v, ks, table = _cache(c, seed)
        q = _randn(_gen(seed, 4), c["batch"], h_q, c["r"], std=2.0)
        st["step"] = tk.prepare_decode(q, k, v, _lens(c, seed), max_ctx=c["ctx"], k_scale=ks, block_table=table,
                                       block_size=c["block"])
    elif c["kind"] == "prefill":
        st["q"], st["k"], st["v"] = _qkv(c, seed)
    elif c["kind"] == "train":
        st["q"], st["k"], st["v"] = _qkv(c, seed)
        st["do"] = _randn(_gen(seed, 5), c["batch"], h_q, c["seq"], d)
    elif c["kind"] == "project":
        x = _randn(_gen(seed, 6), c["batch"], c["seq"], d_model)
        ws = list(zip(_weights(c, seed), (h_q, h_kv, h_kv)))
        if c["seq"] == 1:
            st["steps"] = [tk.prepare_project_heads(x, w, n) for w, n in ws]
        else:
            st["x"], st["ws"] = x, ws
    elif c["kind"] == "append":
        g = _gen(seed, 7)
        st["kn"], st["vn"] = _randn(g, c["batch"], h_kv, c["n_new"], c["r"]), _randn(g, c["batch"], h_kv, c["n_new"], d)
        st["cache"] = _cache(c, seed, empty=True)
        st["pos"] = _starts(c, seed)
    elif c["kind"] == "layer":
        k, v, ks, table = _cache(c, seed)
        x = _randn(_gen(seed, 6), c["batch"], 1, d_model)
        wq, wk, wv = _weights(c, seed)
        lens = _lens(c, seed)
        pq, pk, pv = (tk.prepare_project_heads(x, w, n) for w, n in ((wq, h_q), (wk, h_kv), (wv, h_kv)))
        pa = tk.prepare_cache_append(pk.result, pv.result, lens - 1, k, v, k_scale=ks, block_table=table,
                                     block_size=c["block"])
        pd = tk.prepare_decode(pq.result.view(c["batch"], h_q, c["r"]), k, v, lens, max_ctx=c["ctx"], k_scale=ks,
                               block_table=table, block_size=c["block"])
        st["steps"], st["cache"] = (pq, pk, pv, pa, pd), [t for t in (k, v, ks) if t is not None]
    return st


def _starts(c, seed):
    """First positions written: anywhere that leaves room for the new rows."""
    u = torch.rand(c["batch"], generator=torch.Generator().manual_seed(seed + 31))
    return (u * (c["ctx"] - c["n_new"] + 1)).to(torch.int32).clamp_(max=c["ctx"] - c["n_new"]).cuda()


def run(state):
    st, c = state, state["case"]
    if c["kind"] == "decode":
        return st["step"]()
    if c["kind"] == "prefill":
        return tk.tk_attn_prefill(st["q"], st["k"], st["v"], causal=c["causal"])
    if c["kind"] == "train":
        o, lse = tk.tk_attn_prefill_lse(st["q"], st["k"], st["v"])
        return (o, lse) + tuple(tk.tk_attn_prefill_backward(st["q"], st["k"], st["v"], o, st["do"], lse))
    if c["kind"] == "project":
        if "steps" in st:
            return [step() for step in st["steps"]]
        return [tk.tk_project_heads(st["x"], w, n) for w, n in st["ws"]]
    if c["kind"] == "append":
        k, v, ks, table = st["cache"]
        tk.tk_cache_append(st["kn"], st["vn"], st["pos"], k, v, k_scale=ks, block_table=table, block_size=c["block"])
        return [t for t in (k, v, ks) if t is not None]
    for step in st["steps"]:
        out = step()
    return [out] + st["cache"]


# ------------------------------------------------------------------ what a pass cannot do without


def _visible(c):
    """Visible (query, key) pairs of one head of one sequence."""
    sq = c["seq_q"] if "seq_q" in c else c["seq"]
    sk = c["seq_k"] if "seq_k" in c else c["seq"]
    if not c.get("causal", True):
        return sq * sk
    return sq * (sk - sq) + sq * (sq + 1) // 2


def work(case):
    c = case
    d_model, h_q, h_kv, d = MODELS[c["model"]]
    r, b = c["r"], c["batch"]
    nbytes = flops = 0.0
    if c["kind"] in ("decode", "layer"):
        tokens = b * c["ctx"] * (0.5625 if c.get("ragged") else 1.0)  # the mean of the ragged lengths
        nbytes += tokens * h_kv * (_key_row(c) + 2 * d) + b * h_q * (r + d) * 2
        flops += tokens * h_q * 2 * (r + d)
    if c["kind"] in ("project", "layer"):
        n, cols = b * c.get("seq", 1), h_q * r + h_kv * (r + d)
        nbytes += 2 * (cols * d_model + n * d_model + n * cols)
        flops += 2 * n * d_model * cols
    if c["kind"] in ("append", "layer"):
        nbytes += b * h_kv * c.get("n_new", 1) * (2 * r + 2 * d + _key_row(c) + 2 * d)
    if c["kind"] in ("prefill", "train"):
        size = 4 if c.get("dtype") == "f32" else 2
        sq = c["seq_q"] if "seq_q" in c else c["seq"]
        sk = c["seq_k"] if "seq_k" in c else c["seq"]
        nbytes += size * b * (h_q * sq * (r + d) + h_kv * sk * (r + d))
        flops += 2 * (r + d) * b * h_q * _visible(c)
        if c["kind"] == "train":  # reads dO beside them, writes dQ, dK, dV and the log-sum-exp
            nbytes += 2 * b * (h_q * sq * (r + d) + h_kv * sk * (r + d)) + 4 * b * h_q * sq
            flops += 2 * (3 * r + 2 * d) * b * h_q * _visible(c)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the error against `exact` that was measured at the listed sizes: 3e-7 to 4e-7 in fp32
    and 2e-3 in bf16 (one rounding of each output, and of each probability), 3e-3 for gradients and 4e-3 for a
    layer, whose queries, keys and values are rounded between the calls."""
    if case["kind"] == "append":
        return "exact"
    if case.get("dtype") == "f32":
        return {"rel": 2e-6}
    if case["kind"] == "layer":
        return {"rel": 1.7e-2, "differ": 1e-2}
    return {"rel": 1.2e-2 if case["kind"] == "train" else 9e-3}


# ------------------------------------------------------------------ the same in 64 bits


def _attend(q, k, v, scale, offset=None):
    """softmax(scale q k^T) v and its log-sum-exp for one head's queries [n, r]; row i sees keys 0 .. i + offset."""
    s = torch.matmul(q.double(), k.double().t()) * scale
    if offset is not None:
        s.masked_fill_(torch.ones(s.shape, dtype=torch.bool, device=s.device).triu_(offset + 1), -math.inf)
    lse = torch.logsumexp(s, dim=-1)
    p = s.sub_(lse[:, None]).exp_()
    return torch.matmul(p, v.double()), lse, p


def _exact_decode(c, q, k, v, ks, table, lens):
    _, h_q, h_kv, d = MODELS[c["model"]]
    group = h_q // h_kv
    out = torch.empty(c["batch"], h_q, d, dtype=torch.float64, device="cuda")
    for b, n in enumerate(lens.tolist()):
        if table is not None:
            idx = table[b].long()
            kb, vb = k[idx].transpose(0, 1).flatten(1, 2), v[idx].transpose(0, 1).flatten(1, 2)
            sb = None if ks is None else ks[idx].transpose(0, 1).flatten(1, 2)
        else:
            kb, vb, sb = k[b], v[b], None if ks is None else ks[b]
        for g in range(h_kv):
            kd = _dequantise(kb[g, :n], None if sb is None else sb[g, :n], c["keys"])
            h = slice(g * group, (g + 1) * group)
            out[b, h] = _attend(q[b, h], kd, vb[g, :n], c["r"] ** -0.5)[0]
    return out


def _heads(y, n):
    return y.unflatten(-1, (n, -1)).transpose(1, 2).contiguous()


def exact(case, seed):
    c = case
    d_model, h_q, h_kv, d = MODELS[c["model"]]
    group, scale = h_q // h_kv, c["r"] ** -0.5
    if c["kind"] == "append":
        return None  # bytes, compared as they are
    if c["kind"] == "decode":
        k, v, ks, table = _cache(c, seed)
        q = _randn(_gen(seed, 4), c["batch"], h_q, c["r"], std=2.0)
        return _exact_decode(c, q, k, v, ks, table, _lens(c, seed))
    if c["kind"] == "project":
        x = _randn(_gen(seed, 6), c["batch"], c["seq"], d_model).double()
        return [_heads(torch.matmul(x, w.double().t()), n) for w, n in zip(_weights(c, seed), (h_q, h_kv, h_kv))]
    if c["kind"] == "layer":
        if c["keys"] != "bf16":
            return None  # the new key's code is a rounding, with no value in 64 bits
        k, v, ks, table = _cache(c, seed)
        lens = _lens(c, seed)
        x = _randn(_gen(seed, 6), c["batch"], 1, d_model).double()
        q, kn, vn = (_heads(torch.matmul(x, w.double().t()), n) for w, n in zip(_weights(c, seed), (h_q, h_kv, h_kv)))
        k, v = k.double(), v.double()
        for b, n in enumerate(lens.tolist()):
            at = n - 1
            row = (int(table[b, at // c["block"]]), slice(None), at % c["block"]) if c["paged"] else (b, slice(None), at)
            k[row], v[row] = kn[b, :, 0], vn[b, :, 0]
        return [_exact_decode(c, q[:, :, 0], k, v, ks, table, lens), k, v]
    q, k, v = _qkv(c, seed)
    sq, sk = q.shape[2], k.shape[2]
    offset = sk - sq if c.get("causal", True) else None
    o = torch.empty(c["batch"], h_q, sq, d, dtype=torch.float64, device="cuda")
    if c["kind"] == "prefill":
        for b in range(c["batch"]):
            for h in range(h_q):
                o[b, h] = _attend(q[b, h], k[b, h // group], v[b, h // group], scale, offset)[0]
        return o
    do = _randn(_gen(seed, 5), c["batch"], h_q, c["seq"], d).double()
    lse = torch.empty(c["batch"], h_q, sq, dtype=torch.float64, device="cuda")
    dq, dk, dv = (torch.zeros(t.shape, dtype=torch.float64, device="cuda") for t in (q, k, v))
    for b in range(c["batch"]):
        for h in range(h_q):
            g = h // group
            o[b, h], lse[b, h], p = _attend(q[b, h], k[b, g], v[b, g], scale, offset)
            dv[b, g] += torch.matmul(p.t(), do[b, h])
            ds = torch.matmul(do[b, h], v[b, g].double().t()).sub_((do[b, h] * o[b, h]).sum(-1, keepdim=True)).mul_(p)
            dq[b, h] = torch.matmul(ds, k[b, g].double()) * scale
            dk[b, g] += torch.matmul(ds.t(), q[b, h].double()) * scale
    return o, lse, dq, dk, dv
