"""The calls that the time of an agent simulation goes into, as cases to measure.

Every case is one call, or one short run of calls, that a serving loop makes
through the package's public entry points: decode steps and prefill forwards of
a model (``metro.Model``), and the single operations of ``metro_ops.h``.  The
shapes are those of ``synth`` (Llama-3-8B and 70B layers, the tiny test model)
with the context and prompt lengths of the agents' calls.

A "model" case has few layers (the layers of one model are alike) and, where
the layers are what it is about, a small vocabulary.  Its sequences are forked
from prefilled contexts by page reference and closed again, so that a pass can
be repeated; contexts are whole pages long, which makes the forks host work
only, and a run decodes several tokens, so that last pages are partly filled.
"""

import math

import numpy as np
import torch

from paper_2411_03519_amd import metro, synth

SHAPES = {"tiny": synth.TINY, "8b": synth.LLAMA3_8B, "70b": synth.LLAMA3_70B}
SMALL_VOCAB = synth.TINY["vocab"]
DEV = "cuda"


def listed():
    return [
        # Four agents of the test-sized model: nothing but launches and latency.
        dict(name="tiny_decode", kind="decode", shape="tiny", layers=2, vocab=4096, loaded=True, batch=4, lo=32, hi=128,
             dist="uniform", steps=4),
        # One agent waiting alone for its reply, with the full vocabulary: the latency of a whole call.
        dict(name="8b_decode_1", kind="decode", shape="8b", layers=2, vocab=128256, loaded=False, batch=1, lo=256, hi=4096,
             dist="agents", steps=4),
        # The batch of the benchmark's simulation: 25 agents, contexts around 1200 tokens.
        dict(name="8b_decode_25", kind="decode", shape="8b", layers=2, vocab=4096, loaded=True, batch=25, lo=256, hi=4096,
             dist="agents", steps=4),
        # The median ready batch of the 1000-agent trace.
        dict(name="8b_decode_123", kind="decode", shape="8b", layers=2, vocab=4096, loaded=True, batch=123, lo=256, hi=4096,
             dist="agents", steps=4),
        # A layer of the 70B model at its benchmark batch.
        dict(name="70b_decode_128", kind="decode", shape="70b", layers=1, vocab=4096, loaded=True, batch=128, lo=1024, hi=3072,
             dist="uniform", steps=4),
        # All prompts of 25 agents in one forward: the benchmark's prefill.
        dict(name="8b_prefill_25", kind="prefill", shape="8b", layers=1, vocab=4096, loaded=True, decode=0, chunks=25,
             new_lo=256, new_hi=4096, dist="agents", lo=0, hi=0),
        # The engine's mixed forward: 48 running requests' next tokens and 512-token chunks of four waiting prompts.
        dict(name="8b_mixed", kind="prefill", shape="8b", layers=2, vocab=4096, loaded=True, decode=48, chunks=4,
             new_lo=301, new_hi=512, dist="uniform", lo=256, hi=2048),
        # An agent's next call: a fresh observation of some 160 tokens after a cached preamble and persona.
        dict(name="8b_observation", kind="prefill", shape="8b", layers=2, vocab=4096, loaded=True, decode=0, chunks=1,
             new_lo=161, new_hi=161, dist="uniform", lo=448, hi=448),
        # Decode attention of a few agents with long histories (ragged contexts past many pages).
        dict(name="attn_decode_long", kind="attn_decode", hd=128, nq=32, nkv=8, rows=6, lo=3000, hi=30000),
        # Prefill attention of a long history read in one chunk.
        dict(name="attn_prefill_long", kind="attn_prefill", hd=128, nq=32, nkv=8, items=2, new_lo=3000, new_hi=4096,
             lo=2000, hi=8000),
        # The end of a call on its own: norm, logits over the full vocabulary and the greedy token.
        dict(name="8b_head_64", kind="head", shape="8b", vocab=128256, rows=64),
        # A feed-forward block on an odd number of rows (a large ready batch).
        dict(name="8b_ffn_301", kind="ffn", shape="8b", rows=301),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "mixed", "attn_decode", "attn_prefill",
                       "head", "ffn"])
    if kind == "decode":
        name = rng.choice(["tiny", "8b", "8b", "70b"])
        batch = _log_int(rng, 1, 256 if name == "8b" else 128)
        lo = _log_int(rng, 16, 1024)
        return dict(kind=kind, shape=name, layers=1 if name == "70b" else 2, vocab=SMALL_VOCAB, loaded=True, batch=batch,
                    lo=lo, hi=lo * rng.choice([1, 2, 3]), dist="uniform", steps=rng.choice([2, 3, 4]))
    if kind == "prefill":
        name = rng.choice(["tiny", "8b", "8b", "70b"])
        total = _log_int(rng, 20, 16000 if name == "8b" else 4000)
        chunks = min(_log_int(rng, 1, 16), total)
        new = max(1, total // chunks)
        lo = rng.choice([0, 0, _log_int(rng, 16, 2048)])
        return dict(kind=kind, shape=name, layers=1, vocab=SMALL_VOCAB, loaded=True, decode=0, chunks=chunks, new_lo=new,
                    new_hi=new + new // 2, dist="uniform", lo=lo, hi=2 * lo)
    if kind == "mixed":
        new = _log_int(rng, 17, 512)
        lo = _log_int(rng, 64, 1500)
        return dict(kind="prefill", shape="8b", layers=2, vocab=SMALL_VOCAB, loaded=True, decode=_log_int(rng, 1, 128),
                    chunks=rng.choice([1, 2, 3, 5]), new_lo=new, new_hi=new + new // 3, dist="uniform", lo=lo, hi=2 * lo)
    hd, nkv, group = rng.choice([(128, 8, 4), (128, 8, 4), (128, 8, 8), (64, 2, 2), (64, 8, 4), (128, 4, 1)])
    if kind == "attn_decode":
        lo = _log_int(rng, 20, 20000)
        rows = max(1, min(_log_int(rng, 1, 256), 160000 // lo))
        return dict(kind=kind, hd=hd, nq=nkv * group, nkv=nkv, rows=rows, lo=lo, hi=lo + lo // 2)
    if kind == "attn_prefill":
        new = _log_int(rng, 20, 3000)
        lo = rng.choice([0, _log_int(rng, 16, 8000)])
        return dict(kind=kind, hd=hd, nq=nkv * group, nkv=nkv, items=rng.choice([1, 2, 3]), new_lo=new,
                    new_hi=new + new // 3, lo=lo, hi=lo + lo // 2)
    if kind == "head":
        return dict(kind=kind, shape=rng.choice(["8b", "8b", "70b"]), vocab=128256, rows=_log_int(rng, 1, 256))
    return dict(kind="ffn", shape=rng.choice(["8b", "8b", "70b"]), rows=_log_int(rng, 1, 2000))


# --- sizes ---------------------------------------------------------------------


def _shape(case):
    return dict(SHAPES[case["shape"]], n_layers=case.get("layers", 1), vocab=case["vocab"] if "vocab" in case else SMALL_VOCAB)


def _lengths(n, lo, hi, dist, salt):
    """n lengths of the case (the same for every seed: they are its size)."""
    r = np.random.Generator(np.random.PCG64([n, lo, hi, salt]))
    if dist == "agents":  # the agents' prompts: lognormal, median 1200
        return [int(v) for v in synth.lognormal_lengths(r, n, 1200.0, 0.5, lo, hi)]
    return [int(v) for v in r.integers(lo, hi + 1, n)]


def _contexts(n, lo, hi, dist, salt=1):
    """Context lengths in whole pages."""
    return [max(synth.PAGE if lo else 0, v // synth.PAGE * synth.PAGE) for v in _lengths(n, lo, hi, dist, salt)]


def _items(case):
    """(context before, new tokens) of every sequence of a model case."""
    if case["kind"] == "decode":
        return [(c, case["steps"]) for c in _contexts(case["batch"], case["lo"], case["hi"], case["dist"])]
    d, n = case["decode"], case["chunks"]
    ctx = _contexts(d + n, case["lo"], case["hi"], "uniform")
    return list(zip(ctx, [1] * d + _lengths(n, case["new_lo"], case["new_hi"], case["dist"], 2)))


def _params(shape):
    """(parameters of one layer's matrices, of the head)"""
    d, hd = shape["d_model"], shape["head_dim"]
    qkv = (shape["n_heads"] + 2 * shape["n_kv_heads"]) * hd
    return d * (qkv + shape["n_heads"] * hd + 3 * shape["ffn_dim"]), d * shape["vocab"]


def work(case):
    kind = case["kind"]
    if kind in ("decode", "prefill"):
        s = _shape(case)
        L, (layer, head) = s["n_layers"], _params(s)
        kvb = 2 * s["n_kv_heads"] * s["head_dim"] * 2
        items = _items(case)
        calls = case["steps"] if kind == "decode" else 1
        rows = sum(n for _, n in items)
        heads = rows if kind == "decode" else len(items)
        keys = sum(n * c + n * (n + 1) // 2 for c, n in items)  # (query, key) pairs
        read = keys if kind == "decode" else sum(c for c, _ in items)  # a step reads its context again
        return {"bytes": calls * (L * layer + head) * 2 + L * kvb * (read + rows) + rows * s["d_model"] * 2
                + heads * s["vocab"] * 4,
                "flops": 2 * rows * L * layer + 2 * heads * head + 4 * L * s["n_heads"] * s["head_dim"] * keys}
    if kind in ("attn_decode", "attn_prefill"):
        hd, nq, nkv = case["hd"], case["nq"], case["nkv"]
        items = _attn_items(case)
        keys = sum(n * c + n * (n + 1) // 2 for c, n in items)
        return {"bytes": sum(c + n for c, n in items) * nkv * hd * 4 + 2 * sum(n for _, n in items) * nq * hd * 2,
                "flops": 4 * nq * hd * keys}
    s = _shape(case)
    d, F, m = s["d_model"], s["ffn_dim"], case["rows"]
    if kind == "head":
        return {"bytes": 2 * d * s["vocab"] + m * d * 4 + m * s["vocab"] * 4, "flops": 2 * m * d * s["vocab"]}
    return {"bytes": 2 * 3 * d * F + 2 * m * d * 4, "flops": 6 * m * d * F}


def tolerance(case):
    kind = case["kind"]
    if kind in ("decode", "prefill"):
        return {"rel": 2e-2}  # a changed last bit of fp32 sums grows over the bf16 storage points of one or two layers
    if kind in ("attn_decode", "attn_prefill"):
        return {"rel": 5e-4}  # outputs are bf16: a share of them may round the other way
    if kind == "head":
        return {"rel": 5e-4, "differ": 0.1}  # the norm's output is bf16
    return {"rel": 1e-3}


# --- inputs --------------------------------------------------------------------


def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 16 + salt)
    return g


def _normal(g, shape, std):
    """bf16 normal values, drawn in pieces to bound the float32 memory."""
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 27):
        n = min(1 << 27, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device=DEV).mul_(std)
    return out


def _weights(case, seed):
    """{(name, layer): bf16 tensor} of a model, as a checkpoint would hold them."""
    s, g = _shape(case), _gen(seed)
    names = [("embed", -1), ("final_norm", -1), ("lm_head", -1)]
    names += [(n, layer) for layer in range(s["n_layers"]) for n in synth.LAYER_TENSORS]
    out = {}
    for name, layer in names:
        w = _normal(g, synth.tensor_shape(s, name), 0.1 if name.endswith("norm") else 0.02)
        out[name, layer] = (w.float() + 1.0).to(torch.bfloat16) if name.endswith("norm") else w
    return out


def _tokens(case, seed):
    """(context tokens, new tokens) of every sequence."""
    r = np.random.Generator(np.random.PCG64([seed, 11]))
    v = _shape(case)["vocab"]
    return [(r.integers(0, v, c), r.integers(0, v, n)) for c, n in _items(case)]


GROUP_TOKENS = 8192  # tokens of one forward while contexts are prefilled


def _prepare_model(case, seed):
    s, items = _shape(case), _items(case)
    n, longest = len(items), max(c + k for c, k in items)
    pages = sum(c // synth.PAGE + 2 * (k // synth.PAGE + 2) for c, k in items) + 64
    page_bytes = 2 * s["n_kv_heads"] * synth.PAGE * s["head_dim"] * 2 * s["n_layers"]
    max_tokens = max(GROUP_TOKENS, sum(k for _, k in items) if case["kind"] == "prefill" else 0)
    model = metro.Model(s, max_batch=n, max_tokens=max_tokens, max_context=longest + synth.PAGE, max_seqs=2 * n + 2,
                        kv_pool_bytes=pages * page_bytes, seed=seed)
    if case["loaded"]:
        for (name, layer), w in _weights(case, seed).items():
            model.load_weight(name, layer, w.cpu().view(torch.int16).numpy().view(np.uint16))
    toks = _tokens(case, seed)
    base = [model.seq_open() if c else None for c, _ in items]
    left = [(i, off) for i, (c, _) in enumerate(items) for off in range(0, c, GROUP_TOKENS // 4)]
    left.sort(key=lambda p: p[1])  # one piece of a sequence per forward, in order
    while left:
        now, used, seen = [], 0, set()
        for p in left:
            k = min(GROUP_TOKENS // 4, items[p[0]][0] - p[1])
            if p[0] in seen or used + k > GROUP_TOKENS:
                break
            seen.add(p[0])
            used += k
            now.append(p)
        left = left[len(now):]
        model.prefill_chunk([base[i] for i, _ in now], [toks[i][0][o:o + GROUP_TOKENS // 4] for i, o in now])
    st = dict(case=case, model=model, base=base, ctx=[c for c, _ in items])
    if case["kind"] == "decode":
        feed = np.stack([t for _, t in toks], axis=1).astype(np.int32)
        st["feed"] = [torch.from_numpy(f).to(DEV) for f in feed]
        st["logits"] = [torch.zeros(n, s["vocab"], device=DEV) for _ in feed]
    else:
        st["new"] = [t for _, t in toks]
        st["logits"] = torch.zeros(n, s["vocab"], device=DEV)
    st["next"] = torch.zeros(n, dtype=torch.int32, device=DEV)
    return st


def _attn_items(case):
    """(keys before, queries) of every sequence of an attention case."""
    if case["kind"] == "attn_decode":
        return [(c - 1, 1) for c in _lengths(case["rows"], case["lo"], case["hi"], "uniform", 3)]
    return list(zip(_lengths(case["items"], case["lo"], case["hi"], "uniform", 3),
                    _lengths(case["items"], case["new_lo"], case["new_hi"], "uniform", 4)))


def _attn_inputs(case, seed):
    """q [rows, nq, hd], K and V [pages, nkv, 16, hd] (bf16) and the page ids of the sequences, one after the other."""
    g, items = _gen(seed, 1), _attn_items(case)
    pages = [-(-(c + n) // synth.PAGE) for c, n in items]
    total = sum(pages)
    q = _normal(g, (sum(n for _, n in items), case["nq"], case["hd"]), 1.5)
    k = _normal(g, (total, case["nkv"], synth.PAGE, case["hd"]), 1.0)
    v = _normal(g, (total, case["nkv"], synth.PAGE, case["hd"]), 1.0)
    table = np.random.Generator(np.random.PCG64([seed, 12])).permutation(total).astype(np.int32)
    return items, pages, q, k, v, table


def _prepare_attn(case, seed):
    items, pages, q, k, v, table = _attn_inputs(case, seed)
    P, h, hd = k.shape[0], case["nkv"], case["hd"]
    # the page layout of metro_ops.h
    kt = k.view(P, h, 16, hd // 8, 8).permute(0, 1, 3, 2, 4).reshape(P, 1, h, 16 * hd)
    vt = v.view(P, h, 4, 4, hd // 32, 2, 16).permute(0, 1, 4, 2, 6, 5, 3).reshape(P, 1, h, 16 * hd)
    return dict(case=case, q=q, kv=torch.cat([kt, vt], dim=1).contiguous(), pages=P, table=table,
                cu=np.cumsum([0] + [n for _, n in items]).astype(np.int32),
                before=np.array([c for c, _ in items], np.int32),
                out=torch.zeros(q.shape[0], case["nq"] * hd, dtype=torch.bfloat16, device=DEV))


def _pack(w):
    out = torch.empty_like(w)
    metro.op_pack_weight(w, w.shape[1], w.shape[0], w.shape[1], w.shape[1], out)
    return out


def _block_inputs(case, seed):
    s, g = _shape(case), _gen(seed, 2)
    d, F, m = s["d_model"], s["ffn_dim"], case["rows"]
    x = torch.randn(m, d, generator=g, device=DEV)
    norm = (1.0 + 0.1 * torch.randn(d, generator=g, device=DEV)).to(torch.bfloat16)
    if case["kind"] == "head":
        return s, x, norm, [_normal(g, (s["vocab"], d), 0.02)]
    return s, x, norm, [_normal(g, (F, d), 0.02), _normal(g, (F, d), 0.02), _normal(g, (d, F), 0.02)]


def _prepare_block(case, seed):
    s, x, norm, w = _block_inputs(case, seed)
    d, F, m = s["d_model"], s["ffn_dim"], case["rows"]
    st = dict(case=case, shape=s, x=x, norm=norm, h=torch.zeros(m, d, dtype=torch.bfloat16, device=DEV))
    if case["kind"] == "head":
        st.update(w=_pack(w[0]), logits=torch.zeros(m, s["vocab"], device=DEV),
                  next=torch.zeros(m, dtype=torch.int32, device=DEV))
    else:  # blocks of 8 gate rows and the 8 up rows of the same features
        gu = torch.stack([w[0].view(F // 8, 8, d), w[1].view(F // 8, 8, d)], dim=1).reshape(2 * F, d).contiguous()
        st.update(gu=_pack(gu), down=_pack(w[2]), act=torch.zeros(m, F, dtype=torch.bfloat16, device=DEV),
                  out=torch.zeros(m, d, device=DEV),
                  ws=torch.zeros(8 * m * 2 * F if m <= 512 else 8 * m * d, device=DEV))
    return st


def prepare(case, seed):
    if case["kind"] in ("decode", "prefill"):
        return _prepare_model(case, seed)
    if case["kind"] in ("attn_decode", "attn_prefill"):
        return _prepare_attn(case, seed)
    return _prepare_block(case, seed)


# --- one pass ------------------------------------------------------------------


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind in ("decode", "prefill"):
        m = st["model"]
        seqs = [m.seq_fork(b, c) if c else m.seq_open() for b, c in zip(st["base"], st["ctx"])]
        if kind == "decode":
            for feed, logits in zip(st["feed"], st["logits"]):
                m.decode_step(seqs, feed, logits, st["next"])
        else:
            m.prefill_chunk(seqs, st["new"], st["logits"], st["next"])
        for q in seqs:
            m.seq_close(q)
        return st["logits"]
    if kind == "attn_decode":
        metro.op_attn_decode_noalloc(st["q"], st["kv"], st["pages"], case["nq"], case["nkv"], case["hd"],
                                     st["before"] + 1, st["table"], st["out"])
        return st["out"]
    if kind == "attn_prefill":
        metro.op_attn_prefill(st["q"], st["kv"], st["pages"], case["nq"], case["nkv"], case["hd"], st["cu"],
                              st["before"], st["table"], st["out"])
        return st["out"]
    s, rows = st["shape"], case["rows"]
    d, F = s["d_model"], s["ffn_dim"]
    metro.op_rmsnorm(st["x"], st["norm"], s["rms_eps"], st["h"], rows, d)
    if kind == "head":
        metro.op_gemm(st["h"], st["w"], rows, s["vocab"], d, metro.EPI_STORE_F32, st["logits"], s["vocab"])
        metro.op_argmax(st["logits"], rows, s["vocab"], st["next"])
        return st["logits"], st["next"]
    metro.op_gemm(st["h"], st["gu"], rows, 2 * F, d, metro.EPI_SWIGLU, st["act"], F,
                  workspace=st["ws"] if rows <= 512 else None)
    st["out"].copy_(st["x"])  # the residual that the down projection adds to
    metro.op_gemm(st["act"], st["down"], rows, d, F, metro.EPI_ADD_F32, st["out"], d, workspace=st["ws"])
    return st["act"], st["out"]


# --- the same in float64 -------------------------------------------------------


def _rms(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _rope(x, pos, base):
    half = x.shape[-1] // 2
    th = base ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / (2 * half))
    a = pos[:, None].double() * th
    c, s = torch.cos(a)[:, None], torch.sin(a)[:, None]
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x1 * s + x2 * c], dim=-1)


def _attend(q, k, v, first):
    """q [n, nq, hd] at positions first .. first+n-1 over k, v [keys, nkv, hd]."""
    n, nq, hd = q.shape
    nkv = k.shape[1]
    out = torch.empty_like(q)
    for h in range(nkv):
        for i in range(0, n, 512):
            qi = q[i:i + 512, h * (nq // nkv):(h + 1) * (nq // nkv)]
            keys = first + min(i + 512, n)
            sc = torch.matmul(qi.reshape(-1, hd), k[:keys, h].T.contiguous()).view(qi.shape[0], -1, keys) / math.sqrt(hd)
            pos = first + torch.arange(i, i + qi.shape[0], device=q.device)
            sc.masked_fill_(torch.arange(keys, device=q.device)[None, None] > pos[:, None, None], -math.inf)
            out[i:i + 512, h * (nq // nkv):(h + 1) * (nq // nkv)] = torch.matmul(
                torch.softmax(sc, -1).view(-1, keys), v[:keys, h].contiguous()).view(qi.shape)
    return out


def _exact_model(case, seed):
    s, w = _shape(case), {k: v.double() for k, v in _weights(case, seed).items()}
    hd, eps = s["head_dim"], s["rms_eps"]
    logits = []
    for ctx, new in _tokens(case, seed):
        toks = torch.from_numpy(np.concatenate([ctx, new])).to(DEV)
        pos = torch.arange(len(toks), device=DEV)
        x = w["embed", -1][toks]
        for layer in range(s["n_layers"]):
            p = {n: w[n, layer] for n in synth.LAYER_TENSORS}
            # of the last layer only the rows whose logits are returned are needed
            t0 = len(toks) if layer + 1 < s["n_layers"] else (len(new) if case["kind"] == "decode" else 1)
            h = _rms(x, p["attn_norm"], eps)
            k = _rope((h @ p["wk"].T).view(len(toks), -1, hd), pos, s["rope_base"])
            v = (h @ p["wv"].T).view(len(toks), -1, hd)
            x, h = x[-t0:], h[-t0:]
            q = _rope((h @ p["wq"].T).view(t0, -1, hd), pos[-t0:], s["rope_base"])
            x = x + _attend(q, k, v, len(toks) - t0).reshape(t0, -1) @ p["wo"].T
            h = _rms(x, p["ffn_norm"], eps)
            x = x + (torch.nn.functional.silu(h @ p["wgate"].T) * (h @ p["wup"].T)) @ p["wdown"].T
        logits.append(_rms(x, w["final_norm", -1], eps) @ w["lm_head", -1].T)
    if case["kind"] == "prefill":
        return torch.cat(logits)
    return [torch.stack([r[i] for r in logits]) for i in range(case["steps"])]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("decode", "prefill"):
        if not case["loaded"] or work(case)["flops"] > 4e13 or sum(c for c, _ in _items(case)) > 300_000:
            return None
        return _exact_model(case, seed)
    if kind in ("attn_decode", "attn_prefill"):
        items, pages, q, k, v, table = _attn_inputs(case, seed)
        out, row, at = torch.empty(q.shape[0], case["nq"] * case["hd"], dtype=torch.float64, device=DEV), 0, 0
        for (c, n), p in zip(items, pages):
            ids = torch.from_numpy(table[at:at + p]).long().to(DEV)
            ks, vs = (t[ids].permute(0, 2, 1, 3).reshape(-1, case["nkv"], case["hd"])[:c + n].double() for t in (k, v))
            out[row:row + n] = _attend(q[row:row + n].double(), ks, vs, c).reshape(n, -1)
            row, at = row + n, at + p
        return out
    s, x, norm, w = _block_inputs(case, seed)
    h = _rms(x.double(), norm.double(), s["rms_eps"])
    if kind == "head":
        logits = torch.cat([h @ p.double().T for p in w[0].split(16384)], dim=1)
        return logits, None
    act = torch.nn.functional.silu(h @ w[0].double().T) * (h @ w[1].double().T)
    return act, x.double() + act @ w[2].double().T
