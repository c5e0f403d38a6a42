"""The workloads that this library is timed on, through its public entry points.

The operation is one decoder layer's causal grouped-query attention in two
modes, prefill of a document and continuation over its cached rows, and the
decoder layer around it.  Each listed case is a call that a consumer or a
publisher of cached documents makes:

  decode_rope_call   one new token over a 3774-token document, queries and keys
                     unrotated as the projections leave them, the cache updated
                     in the same call (fp16, host-issued: latency and launches)
  decode_36_layers   one new token through the attention of all 36 layers over
                     16391 cached tokens, captured once as a graph and replayed
                     for each token, as a decode loop does
  continue_24_16k    a 24-token question over a 16384-token document
  continue_q8_24     the same question over an int8 artifact of 30001 tokens
  continue_517_7k    a longer follow-up (517 tokens) over 7001 cached tokens:
                     a retrieved passage appended to a cached document
  prefill_rope_945   a short document's prefill with the rotary embedding
  prefill_32k        the publisher's prefill of a long document
  readers_64         64 questions (24-256 tokens) to one cached 3774-token
                     document in one call
  prefill_d64        prefill at head_dim 64 (16 query heads, 2 kv heads, fp16)
  continue_f32_24    the full-precision path: 24 tokens over 945 cached rows
  layer_24           one whole decoder layer of the 4B geometry: 24 tokens over
                     3774 cached ones
  model_step         one token through a 12-layer stack of the 4B geometry over
                     3774 cached tokens, with the logits (graph-replayed); 12 and
                     not the model's 36 layers, because every layer's 16-bit
                     roundings add up and 36 of them move the logits by 3 %

`draw` gives further calls of the same kinds over the ranges in which they are
used: prefixes of 64 to 32768 rows, 1 to 1024 new tokens, 2 to 64 readers, both
head dims, the three element types, with and without the rotary embedding, the
making of the int8 artifact, and whole layers over the token counts of one
decoding step and of short questions (1, 5, 24 and 40, as the layer's tests).
"""
import math

import torch

from paper_2606_13361_amd import kvr
from paper_2606_13361_amd import kvr_model

DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16, "f32": torch.float32}
ELT = {"bf16": 2, "fp16": 2, "f32": 4}
MODEL = dict(hidden=2560, intermediate=9728, n_q_heads=32, n_kv_heads=8, head_dim=128, eps=1e-6, vocab=151936,
             base=1.0e6)


def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "hq": 32, "hkv": 8, "d": 128, "dtype": "bf16"}
    c.update(kw)
    return c


def listed():
    return [
        _case("decode_rope_call", "continue", entry="rope", L=3774, S=1, dtype="fp16"),
        _case("decode_36_layers", "decode", layers=36, L=16391),
        _case("continue_24_16k", "continue", entry="plain", L=16384, S=24),
        _case("continue_q8_24", "continue_q8", L=30001, S=24),
        _case("continue_517_7k", "continue", entry="plain", L=7001, S=517),
        _case("prefill_rope_945", "prefill", rope=True, L=945),
        _case("prefill_32k", "prefill", rope=False, L=32768),
        _case("readers_64", "readers", rope=False, L=3774, n=64, lo=24, hi=256, lengths=0),
        _case("prefill_d64", "prefill", rope=False, L=2047, hq=16, hkv=2, d=64, dtype="fp16"),
        _case("continue_f32_24", "continue", entry="plain", L=945, S=24, dtype="f32"),
        _case("layer_24", "layer", L=3774, T=24),
        _case("model_step", "model", L=3774, layers=12),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["continue", "continue", "continue", "prefill", "prefill", "readers", "decode", "continue_q8",
                       "quantize", "layer", "model"])
    heads = rng.choice([(32, 8, 128), (32, 8, 128), (32, 8, 128), (8, 8, 128), (12, 3, 128), (64, 8, 128),
                        (16, 2, 64), (8, 2, 64)])
    c = {"kind": kind, "hq": heads[0], "hkv": heads[1], "d": heads[2],
         "dtype": rng.choice(["bf16", "bf16", "fp16", "f32"])}
    f32 = c["dtype"] == "f32"
    if kind == "continue":
        c.update(entry=rng.choice(["plain", "append", "rope"]), L=_log(rng, 64, 4096 if f32 else 32768),
                 S=_log(rng, 1, 64 if f32 else 1024))
    elif kind == "prefill":
        c.update(rope=rng.choice([True, False]), L=_log(rng, 16, 1024 if f32 else 16384))
    elif kind == "readers":
        c.update(rope=rng.choice([True, False]), L=_log(rng, 256, 1024 if f32 else 8192),
                 n=_log(rng, 2, 4 if f32 else 64), lo=24, hi=64 if f32 else 256, lengths=rng.randrange(1 << 20))
    elif kind == "decode":
        c.update(layers=36, L=_log(rng, 256, 1024 if f32 else 16384), hq=32, hkv=8, d=128)
    else:
        c.update(hq=32, hkv=8, d=128, dtype="bf16")
        if kind == "continue_q8":
            c.update(L=_log(rng, 256, 32768), S=_log(rng, 1, 24))
        elif kind == "quantize":
            c.update(L=_log(rng, 256, 32768))
        elif kind == "layer":
            c.update(L=rng.choice([0, _log(rng, 64, 16384), _log(rng, 64, 16384)]), T=rng.choice([1, 5, 24, 40]))
        else:
            c.update(L=_log(rng, 64, 8192), layers=rng.randint(4, 12))
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, shape, dtype, mul=None):
    """N(0, 1) (times mul) in the element type, drawn in fp32."""
    x = torch.randn(shape, generator=g, device="cuda")
    if mul is not None:
        x.mul_(mul)
    return x.to(dtype)


def _lengths(c):
    """Suffix lengths of the readers, uniform on [lo, hi], from the case's own seed."""
    g = torch.Generator()
    g.manual_seed(int(c["lengths"]))
    return torch.randint(c["lo"], c["hi"] + 1, (c["n"],), generator=g).tolist()


def _qkv(g, c, n, dtype):
    return (_randn(g, (n, c["hq"], c["d"]), dtype), _randn(g, (n, c["hkv"], c["d"]), dtype),
            _randn(g, (n, c["hkv"], c["d"]), dtype))


def _layer_weights(g, dtype):
    """One layer's weights: projections N(0, 1/n_in), norm weights 1 + N(0, 0.1^2)."""
    H, I, d = MODEL["hidden"], MODEL["intermediate"], MODEL["head_dim"]
    hq, hkv = MODEL["n_q_heads"], MODEL["n_kv_heads"]

    def mat(o, i):
        return _randn(g, (o, i), dtype, i ** -0.5)

    def vec(n):
        return torch.randn((n,), generator=g, device="cuda").mul_(0.1).add_(1).to(dtype)

    return {"ln1": vec(H), "wqkv": mat((hq + 2 * hkv) * d, H), "q_norm": vec(d), "k_norm": vec(d),
            "wo": mat(H, hq * d), "ln2": vec(H), "wgu": mat(2 * I, H), "wd": mat(H, I)}


def _capacity(c):
    """Cache rows per kv head: what the call fills, rounded up to whole 256-row pages."""
    new = {"continue": c.get("S", 0), "prefill": c["L"], "decode": 1, "layer": c.get("T", 0), "model": 1}.get(c["kind"], 0)
    rows = new if c["kind"] == "prefill" else c["L"] + new
    return (rows + 255) // 256 * 256


def _inputs(c, seed):
    """Every tensor drawn for the case, from the seed alone."""
    g, dt = _gen(seed), DTYPES[c["dtype"]]
    cache = (c["hkv"], _capacity(c), c["d"])
    kind = c["kind"]
    if kind == "prefill":
        return dict(zip("qkv", _qkv(g, c, c["L"], dt)))
    if kind in ("continue", "continue_q8"):
        x = dict(zip("qkv", _qkv(g, c, c["S"], dt)))
        return dict(x, kc=_randn(g, cache, dt), vc=_randn(g, cache, dt))
    if kind == "readers":
        lens = _lengths(c)
        x = dict(zip("qkv", _qkv(g, c, sum(lens), dt)))
        return dict(x, lens=lens, kc=_randn(g, cache, dt), vc=_randn(g, cache, dt))
    if kind == "quantize":
        return dict(kc=_randn(g, cache, dt), vc=_randn(g, cache, dt))
    if kind == "decode":
        n = c["layers"]
        x = dict(zip("qkv", _qkv(g, c, n, dt)))
        kc = torch.empty((n,) + cache, dtype=dt, device="cuda")
        vc = torch.empty_like(kc)
        for i in range(n):
            kc[i] = _randn(g, cache, dt)
            vc[i] = _randn(g, cache, dt)
        return dict(x, kc=kc, vc=vc)
    # a layer, or a stack of them with the output projection
    n = c.get("layers", 1)
    kc = torch.empty((n,) + cache, dtype=dt, device="cuda")
    vc = torch.empty_like(kc)
    layers = []
    for i in range(n):
        layers.append(_layer_weights(g, dt))
        kc[i] = _randn(g, cache, dt)
        vc[i] = _randn(g, cache, dt)
    x = dict(h=_randn(g, (c.get("T", 1), MODEL["hidden"]), dt), layers=layers, kc=kc, vc=vc)
    if kind == "model":
        x["norm"] = torch.randn((MODEL["hidden"],), generator=g, device="cuda").mul_(0.1).add_(1).to(dt)
        x["embed"] = _randn(g, (MODEL["vocab"], MODEL["hidden"]), dt, MODEL["hidden"] ** -0.5)
    return x


# ------------------------------------------------------------------ the calls
def _capture(step):
    """The step as a graph: issued once to load the kernels, then captured."""
    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    return graph


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    dt = DTYPES[c["dtype"]]
    kind, L, d = c["kind"], c["L"], c["d"]
    cap = _capacity(c)
    desc = kvr.make_desc(c["hq"], c["hkv"], d, dt, cap)
    st = dict(x, case=c, desc=desc)
    if "q" in x:
        st["out"] = torch.empty_like(x["q"])
    if kind == "prefill":
        st["kc"] = torch.zeros((c["hkv"], cap, d), dtype=dt, device="cuda")
        st["vc"] = torch.zeros_like(st["kc"])
        if c["rope"]:
            st["rope"] = kvr.RopeTable(d, cap)
    elif kind == "continue":
        if c["entry"] == "rope":
            st["rope"] = kvr.RopeTable(d, cap)
            st["ws"] = kvr.workspace_for_rope(desc, L, c["S"])
        else:
            st["ws"] = kvr.workspace_for(desc, L, c["S"])
    elif kind == "readers":
        st["cu"] = [0]
        for s in x["lens"]:
            st["cu"].append(st["cu"][-1] + s)
        if c["rope"]:
            st["rope"] = kvr.RopeTable(d, cap + c["hi"])
            st["ws"] = kvr.workspace_for_rope(desc, L, st["cu"][-1], c["n"])
        else:
            st["ws"] = kvr.workspace_for(desc, L, st["cu"][-1], c["n"])
    elif kind in ("continue_q8", "quantize"):
        kq, vq, sc = kvr.q8_artifact(desc)
        st.update(kq=kq.zero_(), vq=vq.zero_(), sc=sc)
        if kind == "continue_q8":
            kvr.kvr_quantize_cache(desc, x["kc"], x["vc"], L, kq, vq, sc)
            st["ws"] = kvr.workspace_for(desc, L, c["S"])
            st["kc"] = st["vc"] = None          # the consumer holds the artifact only
    elif kind == "decode":
        st["ws"] = kvr.workspace_for(desc, L, 1)

        def step():
            for i in range(c["layers"]):
                kvr.kvr_continue_append(desc, x["q"][i:i + 1], x["k"][i:i + 1], x["v"][i:i + 1], x["kc"][i], x["vc"][i],
                                        L, 1, st["out"][i:i + 1], st["ws"])
        st["graph"] = _capture(step)
    else:
        T = c.get("T", 1)
        st["rope"] = kvr.RopeTable(d, cap, MODEL["base"])
        st["blas"] = kvr_model.Blas()
        st["ws"] = torch.empty(kvr_model.kvr_layer_workspace_bytes(desc, MODEL, T, L), dtype=torch.uint8, device="cuda")
        st["h_in"] = x["h"]
        st["h"] = x["h"].clone()
        if kind == "model":
            st["xn"] = torch.empty_like(st["h"])
            st["logits"] = torch.empty((1, MODEL["vocab"]), dtype=dt, device="cuda")
            bws = st["ws"][-kvr_model.BLAS_WORKSPACE_BYTES:]

            def step():
                _layers(st, c["layers"], T)
                kvr_model.kvr_rmsnorm(st["h"], st["norm"], MODEL["eps"], st["xn"])
                kvr_model.kvr_linear(st["blas"], st["xn"], st["embed"], st["logits"], ws=bws)
            st["graph"] = _capture(step)
    return st


def _layers(st, n, T):
    L = st["case"]["L"]
    for i in range(n):
        kvr_model.kvr_layer_forward(st["desc"], MODEL, st["layers"][i], st["rope"], st["blas"], st["h"], T, L,
                                    st["kc"][i], st["vc"][i], st["ws"])


def run(state):
    st = state
    c = st["case"]
    kind, L, desc = c["kind"], c["L"], st["desc"]
    if kind == "prefill":
        if c["rope"]:
            kvr.kvr_prefill_rope(desc, st["rope"], st["q"], st["k"], st["v"], L, st["out"], st["kc"], st["vc"])
        else:
            kvr.kvr_prefill(desc, st["q"], st["k"], st["v"], L, st["out"], st["kc"], st["vc"])
        return {"out": st["out"], "kc": st["kc"], "vc": st["vc"]}
    if kind == "continue":
        a = (st["q"], st["k"], st["v"], st["kc"], st["vc"], L, c["S"], st["out"], st["ws"])
        if c["entry"] == "plain":
            kvr.kvr_continue(desc, *a)
            return {"out": st["out"]}
        if c["entry"] == "append":
            kvr.kvr_continue_append(desc, *a)
        else:
            kvr.kvr_continue_rope(desc, st["rope"], *a, append=True)
        return {"out": st["out"], "kc": st["kc"], "vc": st["vc"]}
    if kind == "readers":
        a = (st["q"], st["k"], st["v"], st["cu"], st["kc"], st["vc"], L, st["out"], st["ws"])
        if c["rope"]:
            kvr.kvr_continue_batched_rope(desc, st["rope"], *a)
        else:
            kvr.kvr_continue_batched(desc, *a)
        return {"out": st["out"]}
    if kind == "continue_q8":
        kvr.kvr_continue_q8(desc, st["q"], st["k"], st["v"], st["kq"], st["vq"], st["sc"], L, c["S"], st["out"], st["ws"])
        return {"out": st["out"]}
    if kind == "quantize":
        kvr.kvr_quantize_cache(desc, st["kc"], st["vc"], L, st["kq"], st["vq"], st["sc"])
        return {"kq": st["kq"], "vq": st["vq"], "scales": st["sc"]}
    if kind == "decode":
        st["graph"].replay()
        return {"out": st["out"], "kc": st["kc"], "vc": st["vc"]}
    # the residual stream starts at the tokens' embedding rows
    st["h"].copy_(st["h_in"])
    if kind == "layer":
        _layers(st, 1, c["T"])
        return {"h": st["h"], "kc": st["kc"], "vc": st["vc"]}
    st["graph"].replay()
    return {"logits": st["logits"], "h": st["h"], "kc": st["kc"], "vc": st["vc"]}


# ------------------------------------------------------------------ accounting
def work(case):
    """Each input read once, each output written once; 4 flops per visible
    (query, key) pair and head dim, 2 per weight of a product."""
    c = case
    e, hq, hkv, d, L, kind = ELT[c["dtype"]], c["hq"], c["hkv"], c["d"], c["L"], c["kind"]
    kv, qo = 2 * hkv * d * e, 2 * hq * d * e           # bytes a token: K + V rows, Q + out rows
    pair = 4 * hq * d

    def cont(s, l):
        return s * l + s * (s + 1) // 2

    if kind == "prefill":
        return {"bytes": L * (qo + 2 * kv), "flops": pair * cont(L, 0)}
    if kind == "continue":
        s = c["S"]
        wr = 0 if c["entry"] == "plain" else s * kv
        return {"bytes": L * kv + s * (qo + kv) + wr, "flops": pair * cont(s, L)}
    if kind == "readers":
        lens = _lengths(c)
        return {"bytes": L * kv + sum(lens) * (qo + kv), "flops": pair * sum(cont(s, L) for s in lens)}
    if kind == "decode":
        n = c["layers"]
        return {"bytes": n * (L * kv + qo + 2 * kv), "flops": n * pair * cont(1, L)}
    if kind == "continue_q8":
        s = c["S"]
        return {"bytes": L * kv // 2 + s * (qo + kv), "flops": pair * cont(s, L)}
    if kind == "quantize":
        return {"bytes": L * kv + L * kv // 2, "flops": 2 * L * kv // e}
    H, I = MODEL["hidden"], MODEL["intermediate"]
    params = (hq + 2 * hkv) * d * H + hq * d * H + 3 * I * H
    T, n = c.get("T", 1), c.get("layers", 1)
    b = n * (params * e + (L + T) * kv) + 2 * T * H * e
    f = n * (2 * T * params + pair * cont(T, L))
    if kind == "model":
        b += MODEL["vocab"] * (H + 1) * e
        f += 2 * MODEL["vocab"] * H
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the distance of the present results from 64 bits
    (measured over the listed cases and drawn ones)."""
    if case["kind"] == "quantize":
        return "exact"
    if case["kind"] == "model":
        return {"rel": 3e-2, "max": 0.5}
    if case["kind"] == "layer":
        return {"rel": 1e-2, "max": 0.2}
    return {"bf16": {"rel": 1e-2, "max": 0.3}, "fp16": {"rel": 1.5e-3, "max": 3e-2},
            "f32": {"rel": 6e-6, "max": 1e-4}}[case["dtype"]]


# ------------------------------------------------------------------ 64 bits
def _rotate(x, pos, base=1.0e6):
    """Half-split rotary embedding of x [n, heads, d] at positions pos [n]."""
    d = x.shape[-1]
    i = torch.arange(d // 2, dtype=torch.float64, device=x.device)
    ang = pos.to(torch.float64)[:, None] * (base ** (-2.0 * i / d))[None, :]
    cs, sn = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * cs - b * sn, b * cs + a * sn], -1)


def _attend(q, k, v, kc=None, vc=None):
    """Causal grouped-query attention of rows q [n, hq, d] over cached rows
    kc/vc [hkv, L, d] and their own k/v [n, hkv, d], in 64 bits."""
    n, hq, d = q.shape
    hkv = k.shape[1]
    G = hq // hkv
    out = torch.empty((n, hq, d), dtype=torch.float64, device=q.device)
    L = 0 if kc is None else kc.shape[1]
    step = max(1, min(n, (1 << 27) // (G * (L + n))))
    for g in range(hkv):
        ks, vs = k[:, g].double(), v[:, g].double()
        if L:
            ks, vs = torch.cat([kc[g].double(), ks]), torch.cat([vc[g].double(), vs])
        for t in range(0, n, step):
            rows = q[t:t + step, g * G:(g + 1) * G].double()
            m, e = rows.shape[0], L + min(n, t + step)
            s = (rows.reshape(m * G, d) @ ks[:e].t()).div_(d ** 0.5).view(m, G, e)
            own = torch.arange(e, device=q.device)[None, :] > (L + t + torch.arange(m, device=q.device))[:, None]
            s.masked_fill_(own[:, None, :], -math.inf)
            s = torch.softmax(s, -1).view(m * G, e)
            out[t:t + m, g * G:(g + 1) * G] = (s @ vs[:e]).view(m, G, d)
    return out


def _with_rows(cache, L, rows):
    """The cache [hkv, cap, d] in 64 bits with rows [n, hkv, d] at L.."""
    c = cache.double().clone()
    c[:, L:L + rows.shape[0]] = rows.double().transpose(0, 1)
    return c


def _rms(x, w):
    return x / (x.square().mean(-1, keepdim=True) + MODEL["eps"]).sqrt() * w.double()


def _decoder_layer(h, W, kc, vc, L):
    """(h, new k rows, new v rows) of one decoder layer in 64 bits."""
    hq, hkv, d = MODEL["n_q_heads"], MODEL["n_kv_heads"], MODEL["head_dim"]
    T = h.shape[0]
    pos = L + torch.arange(T, device=h.device)
    qkv = (_rms(h, W["ln1"]) @ W["wqkv"].double().t()).view(T, hq + 2 * hkv, d)
    q = _rotate(_rms(qkv[:, :hq], W["q_norm"]), pos, MODEL["base"])
    k = _rotate(_rms(qkv[:, hq:hq + hkv], W["k_norm"]), pos, MODEL["base"])
    v = qkv[:, hq + hkv:]
    att = _attend(q, k, v, kc[:, :L], vc[:, :L])
    h = h + att.view(T, hq * d) @ W["wo"].double().t()
    g, u = (_rms(h, W["ln2"]) @ W["wgu"].double().t()).chunk(2, -1)
    return h + (g * torch.sigmoid(g) * u) @ W["wd"].double().t(), k, v


def _dequantized(x, L):
    """Rows [0, L) of a cache as the int8 artifact holds them: symmetric codes
    with one fp32 scale, rounded half to even."""
    x = x[:, :L].float()
    s = x.abs().max() / 127.0
    return torch.round(x / s).clamp_(-127, 127).double() * s.double()


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    kind, L = c["kind"], c["L"]
    if kind == "prefill":
        q, k, v = x["q"].double(), x["k"].double(), x["v"].double()
        if c["rope"]:
            pos = torch.arange(L, device=q.device)
            q, k = _rotate(q, pos), _rotate(k, pos)
        zero = torch.zeros((c["hkv"], _capacity(c), c["d"]), dtype=torch.float64, device=q.device)
        return {"out": _attend(q, k, v), "kc": _with_rows(zero, 0, k), "vc": _with_rows(zero, 0, v)}
    if kind == "continue":
        q, k, v = x["q"].double(), x["k"].double(), x["v"].double()
        if c["entry"] == "rope":
            pos = L + torch.arange(c["S"], device=q.device)
            q, k = _rotate(q, pos), _rotate(k, pos)
        out = _attend(q, k, v, x["kc"][:, :L], x["vc"][:, :L])
        if c["entry"] == "plain":
            return {"out": out}
        return {"out": out, "kc": _with_rows(x["kc"], L, k), "vc": _with_rows(x["vc"], L, v)}
    if kind == "readers":
        out, t = [], 0
        for s in x["lens"]:
            q, k, v = (x[n][t:t + s].double() for n in "qkv")
            if c["rope"]:
                pos = L + torch.arange(s, device=q.device)
                q, k = _rotate(q, pos), _rotate(k, pos)
            out.append(_attend(q, k, v, x["kc"][:, :L], x["vc"][:, :L]))
            t += s
        return {"out": torch.cat(out)}
    if kind == "decode":
        out, kc, vc = [], x["kc"], x["vc"]
        for i in range(c["layers"]):
            q, k, v = (x[n][i:i + 1] for n in "qkv")
            out.append(_attend(q, k, v, kc[i, :, :L], vc[i, :, :L]))
            kc[i, :, L], vc[i, :, L] = k[0], v[0]
        return {"out": torch.cat(out), "kc": kc, "vc": vc}      # the cache rows are copies
    if kind == "continue_q8":
        return {"out": _attend(x["q"], x["k"], x["v"], _dequantized(x["kc"], L), _dequantized(x["vc"], L))}
    if kind == "quantize":
        return {"kq": None, "vq": None,
                "scales": torch.stack([x[n][:, :L].double().abs().max() / 127.0 for n in ("kc", "vc")])}
    h, T = x["h"].double(), c.get("T", 1)
    kc, vc = x["kc"].double(), x["vc"].double()
    for i, W in enumerate(x["layers"]):
        h, k, v = _decoder_layer(h, W, kc[i], vc[i], L)
        kc[i, :, L:L + T], vc[i, :, L:L + T] = k.transpose(0, 1), v.transpose(0, 1)
    if kind == "layer":
        return {"h": h, "kc": kc, "vc": vc}
    return {"logits": _rms(h, x["norm"]) @ x["embed"].double().t(), "h": h, "kc": kc, "vc": vc}
