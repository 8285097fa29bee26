"""What the framework's users have it do, as timed cases: the layers of a chunked prefill, whole prefill chunks, the
first-token step and both directions of the KV store, over the model shapes, chunk sizes and prompt lengths of the
repository's workloads (`synth_inputs.SHAPES`, `bench.py`, `sweeps.py`) and a generic small bf16 model with heads of 64.

A case is a dict of plain values, `op` among them:

    attention    cake_op_attention: one layer's queries of a chunk against the paged keys before and inside it
    gateup       cake_op_gemm_swiglu: the feed-forward input product, silu(gate) * up
    down         cake_op_gemm_residual: the feed-forward output product, added into the float32 residual stream
    prefill      Engine.prefill_chunk through `layers` layers; the result is the chunk's K and V of every layer, and
                 the last layer's hold everything that the layers before it did (two layers: one whole block)
    first_token  Engine.first_token through `layers` layers and the head: the logits and the token
    store_write  Engine.write_store: cached KV quantised (or copied) into a pinned store
    store_load   Engine.load_chunk, unthrottled: a pinned store's pages into the cache

The single-layer ops are called through the C ABI (asynchronous, as `kernel_bench` and the library's own prefill run
them); the other calls are the binding's methods with their default arguments, which return when the work is done.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2410_03065_amd as cake
import synth_inputs as si

SMALL_HD64 = si.ModelShape("small-hd64", 16, 2048, 32, 8, 64, 8192, 32000, "bf16", rope_theta=500000.0)
SHAPES = dict(si.SHAPES, **{SMALL_HD64.name: SMALL_HD64})
PREFILL_VOCAB = 32000      # embedding rows of the prefill cases (a chunk reads only its own tokens' rows)
FORMATS = {"raw": cake.STORE_RAW, "int8": cake.STORE_INT8, "int4": cake.STORE_INT4}


def listed():
    return [
        # the smallest call: the first token of the tiny float32 model after its 2048-token prompt; all latency
        {"name": "first_token_tiny", "op": "first_token", "shape": "tiny-f32", "layers": 2, "tokens": 2048, "page": 128},
        # the last 256-token chunk of the tiny float32 workload: the float32 path
        {"name": "prefill_tiny", "op": "prefill", "shape": "tiny-f32", "layers": 2, "begin": 1792, "rows": 256, "page": 128},
        # a serving step's share of a burst request (51 to 324 tokens arrive among the prefix request's chunks)
        {"name": "prefill_burst", "op": "prefill", "shape": "llama3-8b-shape", "layers": 2, "begin": 0, "rows": 137, "page": 256},
        # a middle chunk of the 32K-token benchmark prompt, 1024 tokens at half way
        {"name": "prefill_chunk", "op": "prefill", "shape": "llama3-8b-shape", "layers": 2, "begin": 15360, "rows": 1024, "page": 256},
        # a small bf16 model with heads of 64 (the other head size the framework takes)
        {"name": "prefill_hd64", "op": "prefill", "shape": "small-hd64", "layers": 2, "begin": 1536, "rows": 512, "page": 128},
        # attention alone: the benchmark prompt's last chunk, grouped queries
        {"name": "attention_32k", "op": "attention", "shape": "llama3-8b-shape", "begin": 31744, "rows": 1024, "page": 256},
        # a ragged piece of a multi-head prompt that starts and ends inside a page
        {"name": "attention_ragged", "op": "attention", "shape": "llama2-7b-shape", "begin": 7003, "rows": 509, "page": 256},
        # feed-forward products of the benchmark chunk and of the 512-token chunks of the 7B workload
        {"name": "gateup_1024", "op": "gateup", "shape": "llama3-8b-shape", "rows": 1024},
        {"name": "down_512", "op": "down", "shape": "llama2-7b-shape", "rows": 512},
        # the first output token after the whole 32K-token prompt: weights and cache streamed once, the full vocabulary
        {"name": "first_token_32k", "op": "first_token", "shape": "llama3-8b-shape", "layers": 4, "tokens": 32768, "page": 256},
        # 8-bit store: a computed prefix written out, and a stored chunk brought back
        {"name": "store_write_int8", "op": "store_write", "shape": "llama3-8b-shape", "layers": 4, "tokens": 4096, "page": 256, "format": "int8"},
        {"name": "store_load_int8", "op": "store_load", "shape": "llama3-8b-shape", "layers": 8, "tokens": 1024, "page": 256, "format": "int8"},
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over the logarithm; made odd about half the time."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(hi, v | 1 if rng.random() < 0.5 else v)


def draw(rng):
    op = rng.choice(["prefill", "prefill", "prefill", "attention", "gateup", "down", "first_token", "store_write", "store_load"])
    page = rng.choice([64, 128, 256])
    wide = rng.choice(["llama3-8b-shape", "llama2-7b-shape"])
    if op == "prefill":
        shape = rng.choice(["tiny-f32", "small-hd64", wide])
        if shape == "tiny-f32":
            return {"op": op, "shape": shape, "layers": 2, "begin": rng.randrange(0, 1793), "rows": _spread(rng, 8, 256), "page": page}
        if shape == "small-hd64":
            return {"op": op, "shape": shape, "layers": 2, "begin": rng.randrange(0, 4096), "rows": _spread(rng, 8, 512), "page": page}
        return {"op": op, "shape": shape, "layers": 2, "begin": rng.randrange(0, 15361), "rows": _spread(rng, 8, 1024), "page": page}
    if op == "attention":
        shape = rng.choice([wide, "llama2-70b-shape", "longalpaca-13b-shape"])
        return {"op": op, "shape": shape, "begin": rng.randrange(0, 15361), "rows": _spread(rng, 8, 1024), "page": page}
    if op in ("gateup", "down"):
        return {"op": op, "shape": rng.choice([wide, wide, "longalpaca-13b-shape", "llama2-70b-shape"]), "rows": _spread(rng, 8, 1024)}
    if op == "first_token":
        shape = rng.choice(["tiny-f32", wide, wide])
        most = 2048 if shape == "tiny-f32" else 32768 if shape == "llama3-8b-shape" else 16384
        return {"op": op, "shape": shape, "layers": 2, "tokens": _spread(rng, 64, most), "page": page}
    return {"op": op, "shape": wide, "layers": 4, "tokens": _spread(rng, 64, 4096), "page": page,
            "format": rng.choice(["raw", "int8", "int4"])}


# ------------------------------------------------------------------ inputs
def _shape(case):
    s = SHAPES[case["shape"]]
    if case["op"] == "first_token":
        return s.with_(n_layers=case["layers"])
    return s.with_(n_layers=case.get("layers", 1), vocab=min(s.vocab, PREFILL_VOCAB if case["op"] == "prefill" else 64))


def _pages(case):
    end = case["begin"] + case["rows"] if "begin" in case else case["tokens"]
    return (end + case["page"] - 1) // case["page"]


def _block_table(case, rng):
    """The pages before the call's range lie anywhere in the pool, the pages of the range side by side at its start."""
    n, first = _pages(case), case["begin"] // case["page"] if case["op"] == "prefill" else 0
    return np.concatenate([n - first + rng.permutation(first), np.arange(n - first)]).astype(np.int32)


def prepare(case, seed):
    shape, op = _shape(case), case["op"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    st = {"case": case, "shape": shape}
    if op in ("gateup", "down"):
        # normed activations (unit variance) resp. silu(gate) * up of a random-weight model; weights N(0, 0.02)
        m, d, ff = case["rows"], shape.d_model, shape.ffn
        tiny = shape.with_(n_layers=1, vocab=64, ffn=256)   # the context only lends its streams and workspaces
        st["eng"] = eng = cake.Engine(tiny, None, max_tokens=1024, max_chunk=1024, page_tokens=256, seed=seed)

        def mat(rows, cols, std):
            return (torch.randn(rows, cols, device="cuda", generator=gen) * std).to(torch.bfloat16)
        if op == "gateup":
            st["a"], st["wg"], st["wu"] = mat(m, d, 1.0), mat(ff, d, 0.02), mat(ff, d, 0.02)
            st["out"] = torch.empty(m, ff, device="cuda", dtype=torch.bfloat16)
        else:
            st["a"], st["w"] = mat(m, ff, 0.7), mat(d, ff, 0.02)
            st["out"] = torch.randn(m, d, device="cuda", generator=gen)
            st["x0"] = st["out"].clone()
        return st
    n, page = _pages(case), case["page"]
    st["eng"] = eng = cake.Engine(shape, None, max_tokens=n * page, max_chunk=min(1024, n * page), page_tokens=page,
                                  block_table=_block_table(case, rng), seed=seed, with_head=op == "first_token")
    if op == "prefill":
        st["tokens"] = rng.integers(0, shape.vocab, case["begin"] + case["rows"]).astype(np.int32)
        first = case["begin"] // page
        eng.pool[:, n - first:].normal_(0.0, 1.0, generator=gen)
        if case["begin"] % page:   # the part of the range's first page that an earlier call has written
            k, v = _kv_views(eng.pool[:, 0], shape, page)
            k[:, :, :case["begin"] % page].normal_(0.0, 1.0, generator=gen)
            v[..., :case["begin"] % page].normal_(0.0, 1.0, generator=gen)
    elif op == "store_load" and case["format"] != "raw":
        bits = 8 if case["format"] == "int8" else 4
        codes = rng.integers(0, 256, (n, shape.n_layers, 2, shape.n_kv * page * shape.head_dim * bits // 8), dtype=np.uint8)
        scales = rng.uniform(0.005, 0.03, (n, shape.n_layers, 2, shape.n_kv * page)).astype(np.float32)
        if bits == 8:
            codes[codes == 128] = 0      # the format's codes are -127 .. 127 and, in 4 bits, -7 .. 7
        else:
            codes = np.where(codes & 15 == 8, codes & 240, codes)
            codes = np.where(codes >> 4 == 8, codes & 15, codes)
        st["images"] = np.concatenate([codes, scales.view(np.uint8)], axis=3)
        eng.set_store_int8(st["images"], FORMATS[case["format"]])
    elif op == "store_load":
        words = rng.standard_normal((n, shape.n_layers, 2, shape.n_kv * page * shape.head_dim), dtype=np.float32)
        st["images"] = (words.view(np.uint32) >> 16).astype(np.uint16)
        eng.set_store(st["images"])
    else:
        eng.pool.normal_(0.0, 1.0, generator=gen)
    if op == "attention":
        st["q"] = torch.randn(shape.n_q, case["rows"], shape.head_dim, device="cuda", generator=gen).to(torch.bfloat16)
        st["out"] = torch.empty(case["rows"], shape.n_q * shape.head_dim, device="cuda", dtype=torch.bfloat16)
    if op == "first_token":
        st["tokens"] = rng.integers(0, shape.vocab, case["tokens"]).astype(np.int32)
    return st


def run(st):
    case, eng, op = st["case"], st["eng"], st["case"]["op"]
    lib, ctx = eng.lib, eng.ctx
    if op == "attention":
        rc = lib.cake_op_attention(ctx, st["q"].data_ptr(), st["out"].data_ptr(), 0, case["begin"], case["rows"], ctypes.byref(eng.kv))
    elif op == "gateup":
        rc = lib.cake_op_gemm_swiglu(ctx, st["a"].data_ptr(), st["wg"].data_ptr(), st["wu"].data_ptr(), st["out"].data_ptr(),
                                     case["rows"], st["shape"].ffn, st["shape"].d_model)
    elif op == "down":
        rc = lib.cake_op_gemm_residual(ctx, st["a"].data_ptr(), st["w"].data_ptr(), st["out"].data_ptr(), case["rows"],
                                       st["shape"].d_model, st["shape"].ffn)
    elif op == "prefill":
        eng.prefill_chunk(st["tokens"], case["begin"], case["rows"])
        return {"kv": eng.pool[:, :_pages(case) - case["begin"] // case["page"]]}
    elif op == "first_token":
        token, _, logits = eng.first_token(st["tokens"], want_logits=True)
        return {"token": token, "logits": logits}
    elif op == "store_write":
        return {"store": eng.write_store(case["tokens"], FORMATS[case["format"]])}
    else:
        eng.load_chunk(0, case["tokens"])
        return {"kv": eng.pool}
    if rc != cake.OK:
        raise cake.CakeError(rc, op)
    return {"out": st["out"]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    s, op = _shape(case), case["op"]
    d, ff, hd = s.d_model, s.ffn, s.head_dim
    hq, hkv, e = s.n_q * hd, s.n_kv * hd, s.elem_bytes
    L = s.n_layers
    layer_weights = d * (hq + 2 * hkv) + hq * d + 3 * d * ff
    if op in ("attention", "prefill"):
        r, keys = case["rows"], case["begin"] + case["rows"]
        attn = 4 * hq * (case["begin"] * r + r * (r + 1) // 2)
        if op == "attention":
            return {"bytes": (2 * r * hq + 2 * hkv * keys) * e, "flops": attn}
        return {"bytes": e * (L * (layer_weights + 2 * hkv * (keys + r)) + r * d), "flops": L * (2 * r * layer_weights + attn)}
    if op == "gateup":
        return {"bytes": 2 * (case["rows"] * (d + ff) + 2 * d * ff), "flops": 4 * case["rows"] * d * ff}
    if op == "down":
        return {"bytes": 2 * (case["rows"] * ff + d * ff) + 8 * case["rows"] * d, "flops": 2 * case["rows"] * d * ff}
    if op == "first_token":
        # K and V of the token are cached: no product with W_k and W_v
        weights = L * (layer_weights - 2 * d * hkv) + s.vocab * d
        return {"bytes": e * (weights + L * 2 * hkv * case["tokens"] + d) + 4 * s.vocab,
                "flops": 2 * weights + L * 4 * hq * case["tokens"]}
    n, page = _pages(case), case["page"]
    raw = n * L * 2 * s.n_kv * page * hd * e
    image = raw if case["format"] == "raw" else n * L * 2 * s.n_kv * page * (hd // (1 if case["format"] == "int8" else 2) + 4)
    return {"bytes": raw + image, "flops": 0}


# ------------------------------------------------------------------ what another correct implementation may differ by
def tolerance(case):
    op, f32 = case["op"], _shape(case).dtype == "f32"
    if op in ("store_write", "store_load"):
        return "exact"
    if f32:
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    if op == "prefill":
        return {"rel": 2e-2, "max": 2e-1}      # bf16 activations through a whole block (6e-3 off the 64-bit result)
    if op == "first_token":
        return {"rel": 1e-2, "max": 1e-1, "differ": 0.01}
    if op == "down":
        return {"rel": 1e-5, "max": 1e-3}      # bf16 operands, float32 sums
    if op == "attention":
        return {"rel": 1e-2, "max": 6e-2}      # bf16 probabilities and result (3e-3 off)
    return {"rel": 7e-3, "max": 2e-2}          # one bf16 result from float32 sums (1.7e-3 off)


# ------------------------------------------------------------------ the same in 64 bits
def _kv_views(pages, shape, page):
    """(K [..., head, token, hd], V [..., head, hd, token]) of pages [..., 2 * n_kv * page * hd]."""
    half = shape.n_kv * page * shape.head_dim
    lead = pages.shape[:-1]
    return (pages[..., :half].unflatten(-1, (shape.n_kv, page, shape.head_dim)),
            pages[..., half:].unflatten(-1, (shape.n_kv, shape.head_dim, page)))


def _layer_kv(eng, shape, layer, tokens):
    """K, V [head][token][hd] of tokens 0 .. tokens-1 in float64."""
    n = (tokens + eng.page_tokens - 1) // eng.page_tokens
    phys = torch.from_numpy(eng.block_table_host[:n].astype(np.int64)).cuda()
    k, v = _kv_views(eng.pool[layer, phys], shape, eng.page_tokens)
    k = k.permute(1, 0, 2, 3).flatten(1, 2)[:, :tokens]
    v = v.permute(1, 0, 3, 2).flatten(1, 2)[:, :tokens]
    return k.double(), v.double()


def _attend(q, k, v, begin):
    """q [head][row][hd] at positions begin + row against k, v [kv head][key][hd] -> [row][head * hd]."""
    heads, rows, hd = q.shape
    group = heads // k.shape[0]
    keys = torch.arange(k.shape[1], device=q.device)
    hidden = keys[None, :] > begin + torch.arange(rows, device=q.device)[:, None]
    out = torch.empty(rows, heads * hd, dtype=torch.float64, device=q.device)
    for h in range(heads):
        s = q[h] @ k[h // group].t().contiguous() / math.sqrt(hd)
        s.masked_fill_(hidden, -math.inf)
        out[:, h * hd:(h + 1) * hd] = torch.softmax(s, dim=1) @ v[h // group].contiguous()
    return out


def _norm(x, gain, eps):
    return x * torch.rsqrt((x * x).mean(dim=1, keepdim=True) + eps) * gain.double()


def _rotate(x, begin, theta):
    """x [row][head][hd], adjacent pairs turned by position * theta^(-2 i / hd)."""
    hd = x.shape[2]
    freq = theta ** (-torch.arange(hd // 2, dtype=torch.float64, device=x.device) * 2 / hd)
    ang = (begin + torch.arange(x.shape[0], dtype=torch.float64, device=x.device))[:, None] * freq
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., 0::2], x[..., 1::2]
    return torch.stack([a * c - b * s, a * s + b * c], dim=-1).flatten(2)


def _mul(x, w):
    return x @ w.double().t().contiguous()


def _silu_mlp(h, wg, wu):
    g = _mul(h, wg)
    return g * torch.sigmoid(g) * _mul(h, wu)


def _exact_layers(st, begin, rows, write):
    """The residual stream of tokens begin .. begin+rows-1 through every layer, with K and V of the tokens written to
    the pool's float64 image by `write` (None: they are in the cache already and the cache is only read)."""
    eng, s = st["eng"], st["shape"]
    hq, hkv = s.n_q * s.head_dim, s.n_kv * s.head_dim
    x = eng.embed[torch.from_numpy(st["tokens"][begin:begin + rows].astype(np.int64)).cuda()].double()
    for l, t in enumerate(eng.layer_tensors):
        qkv = _mul(_norm(x, t["attn_norm"], s.rms_eps), t["wqkv"])
        q = _rotate(qkv[:, :hq].reshape(rows, s.n_q, s.head_dim), begin, s.rope_theta).transpose(0, 1)
        if write is None:
            k, v = _layer_kv(eng, s, l, begin + rows)
        else:
            k_new = _rotate(qkv[:, hq:hq + hkv].reshape(rows, s.n_kv, s.head_dim), begin, s.rope_theta).transpose(0, 1)
            v_new = qkv[:, hq + hkv:].reshape(rows, s.n_kv, s.head_dim).transpose(0, 1)
            write(l, k_new, v_new)
            if l + 1 == s.n_layers:
                break
            k, v = _layer_kv(eng, s, l, begin + rows)
            k, v = torch.cat([k[:, :begin], k_new], dim=1), torch.cat([v[:, :begin], v_new], dim=1)
        x = x + _mul(_attend(q, k, v, begin), t["wo"])
        x = x + _mul(_silu_mlp(_norm(x, t["ffn_norm"], s.rms_eps), t["w_gate"], t["w_up"]), t["w_down"])
    return x


def exact(case, seed):
    op = case["op"]
    if op == "store_write":
        return None
    st = prepare(case, seed)
    eng, s = st["eng"], st["shape"]
    if op == "attention":
        k, v = _layer_kv(eng, s, 0, case["begin"] + case["rows"])
        return {"out": _attend(st["q"].double(), k, v, case["begin"])}
    if op == "gateup":
        return {"out": _silu_mlp(st["a"].double(), st["wg"], st["wu"])}
    if op == "down":
        return {"out": st["x0"].double() + _mul(st["a"].double(), st["w"])}
    if op == "first_token":
        x = _exact_layers(st, case["tokens"] - 1, 1, None)
        return {"token": None, "logits": _mul(_norm(x, eng.final_norm, s.rms_eps), eng.lm_head)[0].cpu().numpy()}
    page = case["page"]
    if op == "prefill":
        begin, rows = case["begin"], case["rows"]
        out = eng.pool[:, :_pages(case) - begin // page].double()
        ks, vs = _kv_views(out, s, page)

        def write(l, k_new, v_new):
            for i in range(0, rows):
                p, t = divmod(begin % page + i, page)
                ks[l, p, :, t] = k_new[:, i]
                vs[l, p, :, :, t] = v_new[:, i]
        _exact_layers(st, begin, rows, write)
        return {"kv": out}
    # store_load: value = code * scale, V turned around (raw: the stored bits)
    n, phys = _pages(case), torch.from_numpy(eng.block_table_host.astype(np.int64))
    out = torch.zeros_like(eng.pool, dtype=torch.float64, device="cpu")
    if case["format"] == "raw":
        words = (st["images"].astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        out[:, phys] = torch.from_numpy(words).flatten(2).transpose(0, 1)
        return {"kv": out}
    ks, vs = _kv_views(out, s, page)
    code_bytes = s.n_kv * page * s.head_dim // (1 if case["format"] == "int8" else 2)
    codes, scales = st["images"][..., :code_bytes], st["images"][..., code_bytes:].copy().view(np.float32).astype(np.float64)
    if case["format"] == "int8":
        values = codes.view(np.int8).astype(np.float64)
    else:
        signed = np.arange(16) - 16 * (np.arange(16) > 7)
        values = np.stack([signed[codes & 15], signed[codes >> 4]], axis=-1).reshape(codes.shape[:-1] + (-1,)).astype(np.float64)
    values = values.reshape(n, s.n_layers, 2, s.n_kv, page, s.head_dim) * scales.reshape(n, s.n_layers, 2, s.n_kv, page, 1)
    values = torch.from_numpy(values).transpose(0, 1)
    ks[:, phys] = values[:, :, 0]
    vs[:, phys] = values[:, :, 1].transpose(-1, -2)
    return {"kv": out}
