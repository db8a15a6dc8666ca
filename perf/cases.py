"""The work that a vision-language program gives this library, one call (or one
step of two calls) per case: the Patch Selection Module on the text query, the
Token Selection Module's projections, the token scoring with its selection and
compaction, the prefill attention over what was kept, and the decode attention
over the compacted cache.

The shapes are those of the repository's own workloads: multi-camera prompts of
6 views (256 or 1024 visual tokens each) and 16-128 text tokens, 32/8 or 16/16
heads of 128, batch 1 and a ragged batch of 8, in bf16, E4M3 and (small) fp32.

Kinds of case (the "kind" entry):
  psm     psm_forward: B queries of T tokens
  tsm     tsm_qk from bf16 hidden states of width Dm
  select  select_score_topk with the packed Q, K, V (gather)
  hidden  token_score_topk without copies (all text rows, or the last `rows`
          ones), then gather_hidden: what a program does that prefills from the
          kept hidden states
  step    select_score_topk, then prefill_attn on what it packed
  attn    prefill_attn on packed sequences
  decode  decode_attn, one new token per sample
"""
import math

import torch

import paper_2506_07416_amd as lv

DTYPES = {"bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn, "f32": torch.float32}
ESIZE = {"bf16": 2, "fp8": 1, "f32": 4}


def listed():
    gqa = dict(Hq=32, Hkv=8, D=128)
    cams = dict(N=6, Tv=1024, T=128)
    return [
        # one query: the smallest network of the path, a chain of short launches
        dict(name="psm, one query", kind="psm", B=1, T=128, d=256, heads=4, d_ff=1024, N=6, layers=4),
        # the same module when a server batches its requests
        dict(name="psm, batch 8", kind="psm", B=8, T=128, d=256, heads=4, d_ff=1024, N=6, layers=4),
        # hidden states of one full multi-camera prompt, every view kept
        dict(name="tsm, one prompt", kind="tsm", B=1, **cams, **gqa, Dm=4096, drop=0),
        # eight prompts, 0-4 of 6 views dropped per sample: the largest call of the path
        dict(name="tsm, ragged batch 8", kind="tsm", B=8, **cams, **gqa, Dm=4096, drop=4),
        # the smallest prompt, fp32: what a program runs to check itself against a CPU
        dict(name="step, tiny fp32", kind="step", dtype="f32", B=1, N=2, Tv=64, T=16, Hq=4, Hkv=4, D=64, keep=0.5,
             drop=0),
        # 256 tokens per view, one KV head per query head, 2 of 6 views dropped
        dict(name="step, 6x256 one prompt", kind="step", dtype="bf16", B=1, N=6, Tv=256, T=64, Hq=16, Hkv=16, D=128,
             keep=0.25, drop=2),
        # selection of the full multi-camera prompt at half the tokens
        dict(name="select, one prompt", kind="select", dtype="bf16", B=1, **cams, **gqa, keep=0.5, drop=0),
        # selection of the ragged batch
        dict(name="select, ragged batch 8", kind="select", dtype="bf16", B=8, **cams, **gqa, keep=0.3, drop=4),
        # prefill attention of the compacted prompt (keep ratio 0.5)
        dict(name="attention, 3200 tokens", kind="attn", dtype="bf16", B=1, top=3200, spread=0, **gqa),
        # prefill attention of a ragged E4M3 batch, odd lengths
        dict(name="attention, fp8 batch 8", kind="attn", dtype="fp8", B=8, top=1971, spread=1000, **gqa),
        # one generated token over one compacted prompt
        dict(name="decode, one prompt", kind="decode", dtype="bf16", B=1, top=3217, spread=0, **gqa),
        # one generated token for each sample of the ragged batch
        dict(name="decode, ragged batch 8", kind="decode", dtype="bf16", B=8, top=1988, spread=1200, **gqa),
    ]


# ------------------------------------------------------------------ drawn cases

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng):
    return dict(zip(("Hq", "Hkv", "D"), rng.choice([(32, 8, 128), (32, 8, 128), (16, 8, 128), (16, 16, 128), (16, 2, 128),
                                                   (16, 16, 64), (32, 8, 64), (8, 4, 64)])))


def _prompt(rng, small=False):
    tv = rng.choice([_log(rng, 32, 256 if small else 1024), 64 if small else 256, 196, 256 if small else 1024])
    return dict(N=rng.randint(1, 8 if not small else 4), Tv=tv, T=_log(rng, 8, 64 if small else 192))


def _one(rng):
    kind = rng.choice(["psm", "tsm", "select", "hidden", "step", "attn", "decode"])
    if kind == "psm":
        d = rng.choice([256, 256, 512])
        return dict(kind=kind, B=_log(rng, 1, 24), T=_log(rng, 9, 300), d=d, heads=d // rng.choice([64, 64, 128]),
                    d_ff=d * rng.choice([2, 4]), N=rng.randint(2, 8), layers=rng.choice([2, 4, 4]))
    if kind == "tsm":
        return dict(kind=kind, B=_log(rng, 1, 8), **_prompt(rng), **_heads(rng), Dm=rng.choice([1024, 2048, 4096]),
                    drop=rng.randint(0, 4))
    if kind == "hidden":
        c = dict(kind=kind, dtype="bf16", B=_log(rng, 1, 8), **_prompt(rng), **_heads(rng), keep=rng.choice([0.25, 0.5, 0.7]),
                 drop=rng.randint(0, 3))
        return dict(c, rows=rng.choice([0, 0, 1]), Dm=c["Hq"] * c["D"])
    if kind in ("select", "step"):
        dt = rng.choice(["bf16", "bf16", "fp8", "f32"])
        small = dt == "f32"
        return dict(kind=kind, dtype=dt, B=_log(rng, 1, 2 if small else 8), **_prompt(rng, small), **_heads(rng),
                    keep=rng.choice([0.25, 0.3, 0.5, 0.8]), drop=rng.randint(0, 3))
    dt = rng.choice(["bf16", "bf16", "fp8", "f32"])
    top = _log(rng, 48, 768 if dt == "f32" else 6272)
    return dict(kind=kind, dtype=dt, B=_log(rng, 1, 2 if dt == "f32" else (8 if kind == "attn" else 32)), top=top,
                spread=rng.randint(0, top // 2), **_heads(rng))


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _one(rng)
        if c.get("drop", 0) < c.get("N", 9) and _cost(c) <= most:
            return c


# ------------------------------------------------------------------ sizes

def _dropped(c):
    """Views dropped in each sample (their number follows from the case, which ones from the seed)."""
    if c["B"] == 1:
        return [c["drop"]]
    return [(3 * b + 1) % (c["drop"] + 1) for b in range(c["B"])]


def _kept(c):
    """(visual tokens that survive the view selection, those kept by the token selection) of each sample."""
    vis = [(c["N"] - n) * c["Tv"] for n in _dropped(c)]
    return [(v, min(v, int(math.floor(c["keep"] * v + 1e-6)))) for v in vis]


def _lens(c):
    """Lengths of the packed sequences: the longest is `top`, the others fall towards top - spread."""
    return [c["top"] - (c["spread"] * ((5 * b) % 8)) // 8 for b in range(c["B"])]


def work(c):
    kind = c["kind"]
    if kind == "psm":
        M, d, ff, n = c["B"] * c["T"], c["d"], c["d_ff"], c["N"]
        per_layer = 4 * d * d + 2 * d * ff
        params = c["layers"] * (per_layer + 9 * d + ff) + 3 * d * d + 2 * n * d
        flops = c["layers"] * (2 * M * per_layer + 4 * M * c["T"] * d) + 4 * M * d * n
        return {"bytes": 4 * (M * d + params + c["B"] * n), "flops": flops}
    if kind == "attn":
        L, E = _lens(c), ESIZE[c["dtype"]]
        out = 4 if c["dtype"] == "f32" else 2
        return {"bytes": sum(L) * c["D"] * ((c["Hq"] + 2 * c["Hkv"]) * E + c["Hq"] * out),
                "flops": sum(2 * n * (n + 1) for n in L) * c["D"] * c["Hq"]}
    if kind == "decode":
        L, E = _lens(c), ESIZE[c["dtype"]]
        out = 4 if c["dtype"] == "f32" else 2
        return {"bytes": (sum(L) + c["B"]) * 2 * c["Hkv"] * c["D"] * E + c["B"] * c["Hq"] * c["D"] * (E + out),
                "flops": 4 * (sum(L) + c["B"]) * c["Hq"] * c["D"]}
    B, T, Hq, Hkv, D = (c[k] for k in ("B", "T", "Hq", "Hkv", "D"))
    if kind == "tsm":
        vis = sum((c["N"] - n) * c["Tv"] for n in _dropped(c))
        keys, qs = vis + B * T, B * T
        return {"bytes": 2 * (keys * c["Dm"] + (Hq + Hkv) * D * c["Dm"] + keys * Hkv * D + qs * Hq * D),
                "flops": 2 * c["Dm"] * D * (keys * Hkv + qs * Hq)}
    E = ESIZE[c["dtype"]]
    rows = c.get("rows", 0) or T
    kept = _kept(c)
    nbytes = sum(rows * Hq * D + (v + T) * Hkv * D for v, _ in kept) * E + B * c["N"] * c["Tv"] * 4
    flops = sum(rows * v + rows * (rows + 1) / 2 for v, _ in kept) * 2 * Hq * D
    packed = sum(k + T for _, k in kept)
    if kind == "hidden":
        nbytes += 2 * packed * c["Dm"] * 2
    else:
        nbytes += 2 * packed * (Hq + 2 * Hkv) * D * E
    if kind == "step":
        nbytes += packed * Hq * D * (4 if c["dtype"] == "f32" else 2)
        flops += sum(2 * (k + T) * (k + T + 1) for _, k in kept) * D * Hq
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _encode(x, dtype):
    """Stored tensor and its scale (E4M3: per-tensor scale amax / 448)."""
    if dtype != "fp8":
        return x.to(DTYPES[dtype]), 1.0
    scale = float(x.abs().max()) / 448.0
    return (x / scale).clamp(-448, 448).to(torch.float8_e4m3fn), scale


def _qkv(g, lead, c, dtype):
    """Queries and keys with logits of order 1 and some tokens that draw far more attention than others
    (a direction of each KV head that every query leans to, and that keys hold to a varying degree)."""
    Hq, Hkv, D = c["Hq"], c["Hkv"], c["D"]
    u = _randn(g, Hkv, D)
    u = u / u.norm(dim=-1, keepdim=True)
    lift = math.sqrt(D) ** 0.5 * 1.2
    q = _randn(g, *lead, Hq, D) + lift * u.repeat_interleave(Hq // Hkv, 0)
    k = _randn(g, *lead, Hkv, D) + lift * _randn(g, *lead, Hkv, 1) * u
    v = _randn(g, *lead, Hkv, D)
    return [_encode(x, dtype) for x in (q, k, v)]


def _view_logits(g, c):
    """Confident view logits: the dropped views of each sample at about -4, the others at about 4."""
    B, N = c["B"], c["N"]
    x = 4.0 + 0.5 * _randn(g, B, N)
    order = torch.rand((B, N), generator=g, device="cuda").argsort(dim=1)
    drop = order < torch.tensor(_dropped(c), device="cuda")[:, None]
    return torch.where(drop, -x, x).contiguous()


def _offsets(c):
    return [v * c["Tv"] for v in range(c["N"] + 1)]


def _cu(lens):
    return torch.tensor([0] + lens, device="cuda").cumsum(0).to(torch.int32)


def _psm_params(g, c):
    """Flat fp32 parameters in the order of the C header, as (name, tensor) parts."""
    d, ff, n = c["d"], c["d_ff"], c["N"]
    parts = []

    def gain(name):
        parts.append((name, 1 + 0.1 * _randn(g, d)))

    def bias(name, m):
        parts.append((name, 0.02 * _randn(g, m)))

    def weight(name, rows, cols):
        parts.append((name, _randn(g, rows, cols) / math.sqrt(cols)))

    for i in range(c["layers"]):
        gain("g1%d" % i), bias("b1%d" % i, d), weight("wqkv%d" % i, 3 * d, d), bias("bqkv%d" % i, 3 * d)
        weight("wo%d" % i, d, d), bias("bo%d" % i, d), gain("g2%d" % i), bias("b2%d" % i, d)
        weight("wup%d" % i, ff, d), bias("bup%d" % i, ff), weight("wdn%d" % i, d, ff), bias("bdn%d" % i, d)
    gain("gf"), bias("bf", d)
    parts.append(("lat", _randn(g, n, d)))
    for p in ("q", "k", "v"):
        weight("wc" + p, d, d), bias("bc" + p, d)
    weight("wh", n, d), bias("bh", n)
    return parts


def _raw(c, seed):
    """The inputs alone, on the GPU (prepare adds the outputs and workspaces that a program keeps)."""
    g = _gen(seed)
    kind = c["kind"]
    if kind == "psm":
        return dict(emb=_randn(g, c["B"], c["T"], c["d"]), parts=_psm_params(g, c))
    if kind == "tsm":
        S = c["N"] * c["Tv"] + c["T"]
        x = _randn(g, c["B"], S, c["Dm"]) * torch.exp(0.3 * _randn(g, c["B"], S, 1))
        wq, wk = (_randn(g, c[h] * c["D"], c["Dm"]) / math.sqrt(c["Dm"]) for h in ("Hq", "Hkv"))
        bf = torch.bfloat16
        return dict(x=x.to(bf), wq=wq.to(bf), wk=wk.to(bf), gamma=1 + 0.1 * _randn(g, c["Dm"]), logit=_view_logits(g, c))
    if kind in ("attn", "decode"):
        (q, qs), (k, ks), (v, vs) = _qkv(g, (sum(_lens(c)),), c, c["dtype"])
        s = dict(q=q, k=k, v=v, scales=dict(q_scale=qs, k_scale=ks, v_scale=vs), cu=_cu(_lens(c)))
        if kind == "decode":
            # the new token's rows, under the scales of the cache that they join
            new = [_randn(g, c["B"], c[h], c["D"]) for h in ("Hq", "Hkv", "Hkv")]
            if c["dtype"] == "fp8":
                new = [(x / f).clamp(-448, 448) for x, f in zip(new, (qs, ks, vs))]
            s.update(zip(("q1", "k1", "v1"), (x.to(DTYPES[c["dtype"]]) for x in new)))
            del s["q"]
        return s
    S = c["N"] * c["Tv"] + c["T"]
    (q, qs), (k, ks), (v, vs) = _qkv(g, (c["B"], S), c, c["dtype"])
    s = dict(q=q, k=k, v=v, scales=dict(q_scale=qs, k_scale=ks, v_scale=vs), logit=_view_logits(g, c))
    if kind == "hidden":
        s["x"] = _randn(g, c["B"], S, c["Dm"]).to(torch.bfloat16)
    return s


def _zeros(*shape, dtype):
    if dtype == torch.float8_e4m3fn:
        return torch.zeros(shape, dtype=torch.uint8, device="cuda").view(dtype)
    return torch.zeros(shape, dtype=dtype, device="cuda")


def _token_mask(c, logit):
    S = c["N"] * c["Tv"] + c["T"]
    return lv.patch_select(logit, _offsets(c), S)[1]


def prepare(case, seed):
    c, s = case, _raw(case, seed)
    s["case"] = c
    kind = c["kind"]
    if kind == "psm":
        s["params"] = torch.cat([t.reshape(-1) for _, t in s.pop("parts")])
        n = int(lv.load().litevlm_psm_workspace(c["B"], c["T"], c["d"], c["heads"], c["d_ff"]))
        s["workspace"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        s["out"] = _zeros(c["B"], c["N"], dtype=torch.float32)
        return s
    B, Hq, Hkv, D = (c[k] for k in ("B", "Hq", "Hkv", "D"))
    if kind == "tsm":
        # the gain is folded into the weights once, when a program loads them
        s["wq"], s["wk"] = (lv.tsm_fold_gain(s[w], s["gamma"]) for w in ("wq", "wk"))
        s["mask"] = _token_mask(c, s["logit"])
        S = s["x"].shape[1]
        # rows that the call leaves alone stay zero
        s["q"], s["k"] = (_zeros(B, S, h, D, dtype=torch.bfloat16) for h in (Hq, Hkv))
        return s
    dt = DTYPES[c["dtype"]]
    odt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    if kind == "attn":
        s["out"] = _zeros(sum(_lens(c)), Hq, D, dtype=odt)
        return s
    if kind == "decode":
        s["out"] = _zeros(B, Hq, D, dtype=odt)
        # the bound that a program keeps on the host: the longest prompt and some room to generate
        s["bound"] = max(_lens(c)) + 64
        n = lv.decode_workspace_bytes(dt, B, Hq, Hkv, D, s["bound"])
        s["workspace"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        return s
    S, V = s["q"].shape[1], c["N"] * c["Tv"]
    out = dict(scores=_zeros(B, V, dtype=torch.float32), kept_index=_zeros(B * S, dtype=torch.int32),
               cu_seqlens=_zeros(B + 1, dtype=torch.int32))
    n = lv.workspace_bytes(B, S, V, Hq, Hkv, D, c.get("rows", 0) or None)
    out["workspace"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    if kind == "hidden":
        s["mask"] = _token_mask(c, s["logit"])
        s["packed"] = _zeros(B * S, c["Dm"], dtype=torch.bfloat16)
    else:
        out.update(view_keep=_zeros(B, c["N"], dtype=torch.uint8), n_visual_kept=_zeros(B, dtype=torch.int32),
                   token_keep=_zeros(B, S, dtype=torch.uint8))
        out.update((n, _zeros(B * S, h, D, dtype=dt)) for n, h in (("qc", Hq), ("kc", Hkv), ("vc", Hkv)))
    if kind == "step":
        s["o"] = _zeros(B * S, Hq, D, dtype=odt)
        # what the host knows of the packed lengths without asking the GPU
        s["bound"] = min(V, int(math.floor(c["keep"] * V + 1e-6))) + c["T"]
    s["out"] = out
    return s


# ------------------------------------------------------------------ the calls

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "psm":
        return lv.psm_forward(s["emb"], s["params"], c["heads"], c["d_ff"], c["N"], c["layers"], out=s["out"],
                              workspace=s["workspace"])
    if kind == "tsm":
        q, k = lv.tsm_qk(s["x"], s["mask"], c["N"] * c["Tv"], s["wq"], s["wk"], c["Hq"], c["Hkv"], c["D"], q=s["q"], k=s["k"])
        return {"q": q, "k": k}
    if kind == "attn":
        return lv.prefill_attn(s["q"], s["k"], s["v"], s["cu"], c["top"], out=s["out"], **s["scales"])
    if kind == "decode":
        return lv.decode_attn(s["q1"], s["k1"], s["v1"], s["k"], s["v"], s["cu"], s["bound"], out=s["out"],
                              workspace=s["workspace"], **s["scales"])
    V = c["N"] * c["Tv"]
    if kind == "hidden":
        o = lv.token_score_topk(s["q"], s["k"], None, s["mask"], c["keep"], V, gather=False, out=s["out"],
                                query_rows=c["rows"] or None, **s["scales"])
        packed = lv.gather_hidden(s["x"], o["kept_index"], o["cu_seqlens"], out=s["packed"])
        return {"scores": o["scores"], "kept_index": o["kept_index"], "cu_seqlens": o["cu_seqlens"], "packed": packed}
    o = lv.select_score_topk(s["logit"], _offsets(c), s["q"], s["k"], s["v"], c["keep"], V, out=s["out"], **s["scales"])
    got = {n: o[n] for n in ("scores", "kept_index", "cu_seqlens", "view_keep", "n_visual_kept", "token_keep", "qc", "kc", "vc")}
    if kind == "step":
        got["o"] = lv.prefill_attn(o["qc"], o["kc"], o["vc"], o["cu_seqlens"], s["bound"], out=s["o"], **s["scales"])
    return got


# ------------------------------------------------------------------ the same in 64 bits

def _wide(x, scale=1.0):
    return (x.float() if x.dtype == torch.float8_e4m3fn else x).double() * scale


def _attend(q, k, v, causal):
    """q [n, Hq, D], k, v [m, Hkv, D] in float64, the last query seeing every key."""
    n, Hq, D = q.shape
    m, G = k.shape[0], Hq // k.shape[1]
    o = torch.empty_like(q)
    hide = torch.ones((n, m), dtype=torch.bool, device=q.device).triu(1 + m - n) if causal else None
    for h in range(Hq):
        x = q[:, h].contiguous() @ k[:, h // G].t().contiguous() / math.sqrt(D)
        if causal:
            x.masked_fill_(hide, -math.inf)
        o[:, h] = torch.softmax(x, -1) @ v[:, h // G].contiguous()
    return o


def _exact_psm(c, seed):
    s = _raw(c, seed)
    p = {n: t.double() for n, t in s["parts"]}
    B, T, d, H = c["B"], c["T"], c["d"], c["heads"]
    ln = lambda x, g, b: torch.nn.functional.layer_norm(x, (d,), p[g], p[b], 1e-5)  # noqa: E731
    h = s["emb"].double().reshape(B * T, d)
    for i in range(c["layers"]):
        qkv = (ln(h, "g1%d" % i, "b1%d" % i) @ p["wqkv%d" % i].t() + p["bqkv%d" % i]).reshape(B, T, 3, H, d // H)
        a = torch.stack([_attend(x[:, 0], x[:, 1], x[:, 2], False) for x in qkv]).reshape(B * T, d)
        h = h + a @ p["wo%d" % i].t() + p["bo%d" % i]
        u = torch.nn.functional.gelu(ln(h, "g2%d" % i, "b2%d" % i) @ p["wup%d" % i].t() + p["bup%d" % i])
        h = h + u @ p["wdn%d" % i].t() + p["bdn%d" % i]
    x = ln(h, "gf", "bf")
    q = p["lat"] @ p["wcq"].t() + p["bcq"]
    k, v = ((x @ p["wc" + n].t() + p["bc" + n]).reshape(B, T, d) for n in ("k", "v"))
    w = torch.softmax(torch.einsum("nd,btd->bnt", q, k) / math.sqrt(d), -1)
    return torch.einsum("bnt,btd,nd->bn", w, v, p["wh"]) + p["bh"]


def _exact_tsm(c, seed):
    s = _raw(c, seed)
    B, V, D = c["B"], c["N"] * c["Tv"], c["D"]
    S = V + c["T"]
    keep = _mask64(c, s["logit"])
    ang = (10.0 ** 6) ** (-2 * torch.arange(D // 2, device="cuda", dtype=torch.float64) / D)

    def project(x, w, H, pos):
        # the folded weights are stored in bf16
        wf = (w.float() * s["gamma"]).to(torch.bfloat16).double()
        y = x.double()
        y = (y @ wf.t() * torch.rsqrt(y.square().mean(-1, keepdim=True) + float(torch.tensor(1e-5)))).reshape(-1, H, D)
        a = (pos.double()[:, None] * ang)[:, None]
        lo, hi = y[..., :D // 2], y[..., D // 2:]
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)

    q, k = (torch.zeros((B, S, c[h], D), dtype=torch.float64, device="cuda") for h in ("Hq", "Hkv"))
    for b in range(B):
        at = keep[b].nonzero()[:, 0]
        pos = torch.arange(at.numel(), device="cuda")
        k[b, at] = project(s["x"][b, at], s["wk"], c["Hkv"], pos)
        q[b, V:] = project(s["x"][b, V:], s["wq"], c["Hq"], pos[-c["T"]:])
    return {"q": q, "k": k}


def _mask64(c, logit):
    keep = (torch.sigmoid(logit.double()) > 0.5).repeat_interleave(c["Tv"], 1)
    return torch.cat([keep, torch.ones((c["B"], c["T"]), dtype=torch.bool, device="cuda")], 1)


def _scores64(c, q, k, keep, rows):
    V, T, G = c["N"] * c["Tv"], c["T"], c["Hq"] // c["Hkv"]
    out = torch.full((c["B"], V), -math.inf, dtype=torch.float64, device="cuda")
    hide = torch.ones((T, T), dtype=torch.bool, device="cuda").triu(1)[T - rows:]
    for b in range(c["B"]):
        at = keep[b].nonzero()[:, 0]
        mass = 0.0
        for h in range(c["Hq"]):
            x = q[b, V + T - rows:, h].contiguous() @ k[b, at, h // G].t().contiguous() / math.sqrt(c["D"])
            x[:, -T:].masked_fill_(hide, -math.inf)
            mass = mass + torch.softmax(x, -1).sum(0)
        out[b, at[:-T]] = mass[:-T] / (c["Hq"] * rows)
    return out


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind == "psm":
        return _exact_psm(c, seed)
    if kind == "tsm":
        return _exact_tsm(c, seed)
    s = _raw(c, seed)
    k, v = (_wide(s[n], s["scales"][n + "_scale"]) for n in ("k", "v"))
    if kind in ("attn", "decode"):
        cu = [0] + torch.tensor(_lens(c)).cumsum(0).tolist()
        spans = list(zip(cu, cu[1:]))
        if kind == "attn":
            q = _wide(s["q"], s["scales"]["q_scale"])
            return torch.cat([_attend(q[a:e], k[a:e], v[a:e], True) for a, e in spans])
        q1, k1, v1 = (_wide(s[n + "1"], s["scales"][n + "_scale"]) for n in "qkv")
        return torch.cat([_attend(q1[b:b + 1], torch.cat([k[a:e], k1[b:b + 1]]), torch.cat([v[a:e], v1[b:b + 1]]), False)
                          for b, (a, e) in enumerate(spans)])
    q = _wide(s["q"], s["scales"]["q_scale"])
    keep = _mask64(c, s["logit"])
    sc = _scores64(c, q, k, keep, c.get("rows", 0) or c["T"])
    got = {"scores": sc}
    if kind == "step":
        V, S = c["N"] * c["Tv"], q.shape[1]
        o = torch.zeros((c["B"] * S, c["Hq"], c["D"]), dtype=torch.float64, device="cuda")
        row = 0
        for b, (_, kb) in enumerate(_kept(c)):
            at = torch.cat([sc[b].argsort(descending=True, stable=True)[:kb].sort().values, torch.arange(V, S, device="cuda")])
            o[row:row + at.numel()] = _attend(q[b, at], k[b, at], v[b, at], True)
            row += at.numel()
        got["o"] = o
    return got


def tolerance(c):
    # About four times the error against exact() that the stored types give: 32-bit sums; bf16
    # outputs and bf16 probabilities; E4M3 probabilities; a bf16 network of a few layers.
    kind, dt = c["kind"], c.get("dtype")
    if kind == "psm":
        return {"rel": 2e-2}
    if kind == "tsm":
        return {"rel": 8e-3}
    differ = {"differ": 0.01} if kind in ("select", "hidden", "step") else {}
    if kind in ("select", "hidden") or dt == "f32":
        return dict(rel=2e-5 if dt == "fp8" else 1e-5, **differ)
    if dt == "fp8" and kind != "decode":
        return dict(rel=0.03, **differ)
    return dict(rel=1e-2, **differ)
