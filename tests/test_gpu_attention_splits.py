"""Attention kernels whose keys may be divided among workgroups, through cake_op_attention against the oracle: the
edges of query and key tiles, short and long prefixes (one key range and many), grouped queries, both head sizes,
and values that a query must not see."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import store as ostore
from oracle import transformer as otf

pytestmark = pytest.mark.gpu


def _case(kind, hd, n_q, n_kv, tok_begin, rows, pt, seed=0, attn_variant=0):
    """(engine, q on the GPU, q / K / V as the kernel sees them in float64)."""
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("attn-splits", 1, 256, n_q, n_kv, hd, 512, 64, kind, rope_theta=500000.0)
    T = tok_begin + rows
    n_log = (T + pt - 1) // pt
    bt = np.random.default_rng(3).permutation(n_log).astype(np.int32)
    eng = cake.Engine(shape, None, max_tokens=n_log * pt, max_chunk=min(1024, n_log * pt), page_tokens=pt, block_table=bt)
    eng.set_tuning(attn_variant=attn_variant)
    rng = np.random.default_rng(seed + rows)
    cache = otf.KVCache(1, T, n_kv, hd)
    cache.k[0] = otf.round_storage(rng.standard_normal((T, n_kv, hd)) * 1.5, kind)
    cache.v[0] = otf.round_storage(rng.standard_normal((T, n_kv, hd)), kind)
    eng.set_store(ostore.pack_store(cache, pt, kind))
    eng.load_chunk(0, T)
    q = otf.round_storage(rng.standard_normal((rows, n_q, hd)), kind)
    Q = torch.from_numpy(q.transpose(1, 0, 2).astype(np.float32).copy()).cuda().to(eng.tdtype)
    return eng, Q, q, cache.k[0], cache.v[0]


def _check(kind, eng, Q, q, k, v, tok_begin, tol):
    rows, n_q, hd = q.shape
    got = eng.op_attention(Q, 0, tok_begin).float().cpu().numpy().reshape(rows, n_q, hd)
    want = otf.attention(q, k, v, np.arange(tok_begin, tok_begin + rows), np.arange(tok_begin + rows))
    err = float(np.abs(got - want).max() / np.abs(want).max())
    print("attention %s: largest error %.2e of the largest value" % (kind, err))
    assert err < tol, err


# float32: a score is a sum of hd products (error below hd * 2^-24 of a magnitude of at most about 30 here), it acts
# in the exponent, and the result is a weighted mean: 64 * 6e-8 * 5 = 2e-5
@pytest.mark.parametrize("hd,n_q,n_kv", [(64, 4, 4), (128, 8, 2)])
@pytest.mark.parametrize("tok_begin,rows,pt", [(0, 1, 64), (0, 33, 64), (31, 32, 64), (300, 95, 128), (1792, 256, 128), (6001, 7, 256)])
def test_attention_f32(hd, n_q, n_kv, tok_begin, rows, pt):
    _check("f32", *_case("f32", hd, n_q, n_kv, tok_begin, rows, pt), tok_begin, 2e-5)


def _poisoned(kind, hd, n_q, n_kv, tok_begin, rows, pt, bad_row, tol):
    """A NaN in V of row `bad_row` of the chunk, and NaNs in the page slots past its last token: the rows before
    `bad_row` are unaffected, it and the rows after it become NaN."""
    import torch
    eng, Q, q, k, v = _case(kind, hd, n_q, n_kv, tok_begin, rows, pt)
    T = tok_begin + rows
    pages = eng.pool[0].view(eng.kv.n_physical_pages, 2, -1)
    bt = eng.block_table_host
    vt = pages[:, 1].view(-1, n_kv, hd, pt)
    p, t = divmod(tok_begin + bad_row, pt)
    vt[int(bt[p]), :, 0, t] = float("nan")
    if T % pt:
        vt[int(bt[T // pt]), :, :, T % pt:] = float("nan")
        pages[:, 0].view(-1, n_kv, pt, hd)[int(bt[T // pt]), :, T % pt:] = float("inf")
    torch.cuda.synchronize()
    got = eng.op_attention(Q, 0, tok_begin).float().cpu().numpy().reshape(rows, n_q, hd)
    want = otf.attention(q, k, v, np.arange(tok_begin, T), np.arange(T))
    clean = got.copy()
    clean[bad_row:, :, 0] = want[bad_row:, :, 0]
    assert np.isnan(got[bad_row:, :, 0]).all()
    assert float(np.abs(clean - want).max() / np.abs(want).max()) < tol


def test_attention_f32_hidden_values_do_not_leak():
    _poisoned("f32", 64, 4, 2, 200, 77, 128, 50, 2e-5)


# Probabilities down to e^-80, one to an element of the result: scores, their differences and V are exact, so a value
# carries the error of the exponentials that formed it (against the tile's reference and, merged, against the row's: 2^-23
# each) and of six roundings in products, sums and the division: 10 * 2^-24.
@pytest.mark.parametrize("first", [1, 40, 300])      # the reference's key in the same tile, another one, another key range
def test_attention_f32_small_probabilities(first):
    import torch
    import paper_2410_03065_amd as cake
    T, hd = 600, 64
    eng = cake.Engine(si.ModelShape("attn-exp", 1, 256, 4, 4, hd, 512, 64, "f32"), None, max_tokens=640, max_chunk=64, page_tokens=64)
    x = (np.round(np.linspace(2.0, 80.0, hd - 1) * 1024) / 1024).astype(np.float32)   # differences of scores are exact too
    cache = otf.KVCache(1, T, 4, hd)
    cache.k[0], cache.v[0] = 0.0, 0.0
    cache.k[0][:, :, 0] = -1000.0
    cache.k[0][0, :, 0] = 0.0                                             # probability 1 before the division, V = 0
    cache.k[0][first:first + hd - 1, :, 0] = -x[:, None]
    for j in range(hd - 1):
        cache.v[0][first + j, :, j] = 1.0
    eng.set_store(ostore.pack_store(cache, 64, "f32"))
    eng.load_chunk(0, T)
    q = torch.zeros(4, 1, hd, device="cuda")
    q[..., 0] = 8.0                                                       # 8 / sqrt(64) = 1
    torch.cuda.synchronize()
    got = eng.op_attention(q, 0, T - 1).cpu().numpy().astype(np.float64).reshape(4, hd)[:, :hd - 1]
    want = np.exp(-x.astype(np.float64)) / (1.0 + np.exp(-x.astype(np.float64)).sum())
    err = float(np.abs(got / want - 1.0).max())
    print("largest relative error %.2e" % err)
    assert err < 10 * 2.0 ** -24, err


# bf16, heads of 64: the scores and the probabilities keep float32's precision (24 bits in the second product), so what
# is left is the rounding of the result to 8 significant bits (in [1, 2) the values lie 2^-7 apart: at most half of
# that, 2^-8 of a value), and 2^-15 for the probabilities and the sums
@pytest.mark.parametrize("n_q,n_kv", [(4, 4), (8, 2), (16, 8)])
@pytest.mark.parametrize("tok_begin,rows,pt", [(0, 1, 64), (0, 33, 64), (63, 32, 64), (64, 65, 128), (300, 95, 128), (1000, 256, 128),
                                               (6001, 7, 256), (4000, 129, 256)])
def test_attention_bf16_hd64(n_q, n_kv, tok_begin, rows, pt):
    _check("bf16", *_case("bf16", 64, n_q, n_kv, tok_begin, rows, pt), tok_begin, 2.0 ** -8 + 2.0 ** -15)


def test_attention_bf16_hd64_hidden_values_do_not_leak():
    _poisoned("bf16", 64, 4, 2, 200, 77, 128, 50, 2.0 ** -8 + 2.0 ** -15)


def test_attention_bf16_hd64_probabilities_keep_float32s_bits():
    """Keys of scores 0, -a and -a - c, c from 2^-10, with V = 0, 1 and -1: the result is the difference of two
    probabilities, 2^-11 of them, so an error of theirs comes out 2^11 times as large.  Float32 exponentials leave 2^-23 of
    each, in all 2^-11 of the result, which is then rounded to bf16 (8 significant bits: 2^-8 of a value at most);
    probabilities of 16 bits are up to 2^-7 off before that."""
    import torch
    import paper_2410_03065_amd as cake
    T, rows, hd = 400, 128, 64
    eng = cake.Engine(si.ModelShape("attn-bits", 1, 256, 4, 4, hd, 512, 64, "bf16"), None, max_tokens=448, max_chunk=128, page_tokens=64)
    cache = otf.KVCache(1, T, 4, hd)
    cache.k[0], cache.v[0] = 0.0, 0.0
    a = 0.30078125
    cache.k[0][:, :, 0] = -1024.0
    cache.k[0][3, :, 0], cache.k[0][170, :, 0], cache.k[0][60, :, 0] = -a, -a, 0.0
    cache.k[0][170, :, 1] = -1.0
    cache.v[0][3], cache.v[0][170] = 1.0, -1.0
    eng.set_store(ostore.pack_store(cache, 64, "bf16"))
    eng.load_chunk(0, T)
    c = 2.0 ** -10 * (1.0 + np.arange(rows) / 128.0)                      # bf16 values
    q = torch.zeros(4, rows, hd)
    q[..., 0], q[..., 1] = 8.0, torch.from_numpy(8.0 * c).float()         # scores -a, -a - c and 0, by 1 / sqrt(64)
    q = q.cuda().to(torch.bfloat16)
    torch.cuda.synchronize()
    got = eng.op_attention(q, 0, T - rows).float().cpu().numpy().reshape(rows, 4 * hd)
    want = ((np.exp(-a) - np.exp(-a - c)) / (1.0 + np.exp(-a) + np.exp(-a - c)))[:, None]
    err = float(np.abs(got / want - 1.0).max())
    print("largest relative error %.2e" % err)
    assert err < 2.0 ** -8 + 2.0 ** -11, err


def test_attention_bf16_hd64_visible_infinities():
    """Infinities in V at keys that the queries see: a query's result is that infinity in that element, a NaN where two of
    opposite sign meet, and every other element is what it would be."""
    import torch
    begin, rows, pt, n_q, n_kv = 900, 70, 128, 8, 2
    eng, Q, q, k, v = _case("bf16", 64, n_q, n_kv, begin, rows, pt)
    vt = eng.pool[0].view(eng.kv.n_physical_pages, 2, -1)[:, 1].view(-1, n_kv, 64, pt)
    where = [(3, 0, 5, np.inf), (130, 0, 6, -np.inf), (517, 1, 7, np.inf), (518, 1, 8, np.inf), (700, 1, 8, -np.inf),
             (910, 0, 9, -np.inf)]                                        # key, KV head, element; the last among the chunk's own
    for key, g, e, x in where:
        vt[int(eng.block_table_host[key // pt]), g, e, key % pt] = x
    torch.cuda.synchronize()
    got = eng.op_attention(Q, 0, begin).float().cpu().numpy().reshape(rows, n_q, 64)
    finite = otf.attention(q, k, v, np.arange(begin, begin + rows), np.arange(begin + rows))
    want = finite.copy()
    for row in range(rows):
        for h in range(n_q):
            for e in range(64):
                hit = [x for key, g, el, x in where if g == h // (n_q // n_kv) and el == e and key <= begin + row]
                if hit:
                    want[row, h, e] = np.nan if len(set(hit)) == 2 else hit[0]
    hit = ~np.isfinite(want)
    assert np.array_equal(got[hit], want[hit], equal_nan=True)
    assert np.isfinite(got[~hit]).all()
    assert float(np.abs(got[~hit] - want[~hit]).max() / np.abs(finite).max()) < 2.0 ** -8 + 2.0 ** -15


# bf16, heads of 128: the result, each probability and the scaled query are rounded to bf16; 2^-7 of the largest value
# covers the three (tests/test_gpu_ops.py::test_attention).  Query heads of a KV head are laid side by side, so a tile of
# queries ends inside a row's heads (r = 3) and a workgroup's rows inside a key tile.
@pytest.mark.parametrize("n_q,n_kv", [(4, 4), (6, 2), (32, 8), (8, 1)])
@pytest.mark.parametrize("tok_begin,rows,pt", [(0, 1, 64), (0, 33, 64), (63, 32, 64), (300, 95, 128), (1000, 256, 128), (6001, 7, 256),
                                               (4000, 129, 256), (9000, 43, 64)])
def test_attention_bf16_hd128(n_q, n_kv, tok_begin, rows, pt):
    _check("bf16", *_case("bf16", 128, n_q, n_kv, tok_begin, rows, pt), tok_begin, 2.0 ** -7)


@pytest.mark.parametrize("kind,hd,n_q,n_kv", [("bf16", 128, 8, 2), ("bf16", 128, 8, 8), ("bf16", 64, 8, 2), ("f32", 64, 4, 4)])
def test_attention_of_a_model_of_few_heads_does_not_depend_on_the_step(kind, hd, n_q, n_kv):
    """Rows computed in one call, in pieces of 128, 64 and 32 and at another length of the prefix: the same bits (a
    prompt's KV must not show where the compute side's last claim ended)."""
    import torch
    begin, rows = 3072, 512
    eng, Q, *_ = _case(kind, hd, n_q, n_kv, begin, rows, 128)
    whole = eng.op_attention(Q, 0, begin)
    for piece in (256, 128, 64, 32):
        for r in range(0, rows, piece):
            q = Q[:, r:r + piece].contiguous()
            torch.cuda.synchronize()
            part = eng.op_attention(q, 0, begin + r)
            assert torch.equal(part, whole[r:r + piece]), (piece, r)


def _prefill_in_steps(eng, toks, steps):
    """The pool after a prefill in steps of the given numbers of tokens, taken in turn until the prompt is through."""
    import torch
    eng.clear_pool()
    at, i = 0, 0
    while at < len(toks):
        n = min(steps[i % len(steps)], len(toks) - at)
        eng.prefill_chunk(toks, at, n)
        at, i = at + n, i + 1
    torch.cuda.synchronize()
    return eng.pool.clone()


@pytest.mark.parametrize("n_q,n_kv,hd,d,ffn", [(4, 4, 64, 256, 688), (8, 2, 64, 512, 1376), (20, 4, 64, 640, 1024), (6, 2, 128, 768, 2056)])
def test_f32_prefill_does_not_depend_on_its_steps(n_q, n_kv, hd, d, ffn):
    """A float32 model's KV has the same bits whatever steps the prompt is computed in: whole chunks, pieces that end
    inside a key tile and a 32-row block, a first step shorter than a key tile."""
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("f32-steps", 2, d, n_q, n_kv, hd, ffn, 128, "f32", rope_theta=500000.0)
    eng = cake.Engine(shape, None, max_tokens=2048, max_chunk=1024, page_tokens=128, seed=3)
    toks = si.make_tokens(1500, shape.vocab, seed=7)
    whole = _prefill_in_steps(eng, toks, [1024])
    for steps in ([512], [256], [7, 101, 300], [37], [33, 1, 950]):
        assert torch.equal(_prefill_in_steps(eng, toks, steps), whole), steps


@pytest.mark.parametrize("hd,n_q,n_kv", [(128, 8, 2), (128, 6, 2), (64, 8, 2), (64, 16, 16)])
def test_attention_of_a_model_of_few_heads_in_ragged_pieces(hd, n_q, n_kv):
    """Pieces that end inside a wave's queries, on both sides of the first key range's end."""
    import torch
    begin, rows = 700, 700
    eng, Q, *_ = _case("bf16", hd, n_q, n_kv, begin, rows, 128)
    whole = eng.op_attention(Q, 0, begin)
    for piece in (101, 37, 450):
        for r in range(0, rows, piece):
            q = Q[:, r:r + piece].contiguous()
            torch.cuda.synchronize()
            assert torch.equal(eng.op_attention(q, 0, begin + r), whole[r:r + piece]), (piece, r)


# Contexts whose bf16 products add up in one order for every step they can have: narrow models, and steps of one tile of
# rows.  few_rows: K ranges are left by the kernel for few rows, as many for a short step as for the longest.
@pytest.mark.parametrize("hd,n_q,n_kv,d,ffn,max_chunk,few_rows", [
    (64, 20, 4, 1280, 3456, 512, False), (64, 32, 8, 2048, 3072, 256, False), (64, 32, 8, 2048, 8192, 128, True),
    (128, 24, 8, 3072, 8192, 128, True), (128, 8, 2, 1024, 2816, 256, False), (64, 8, 8, 512, 1408, 512, False)])
def test_bf16_prefill_of_a_step_free_context_does_not_depend_on_its_steps(hd, n_q, n_kv, d, ffn, max_chunk, few_rows):
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("bf16-steps", 2, d, n_q, n_kv, hd, ffn, 128, "bf16", rope_theta=500000.0)
    eng = cake.Engine(shape, None, max_tokens=2048, max_chunk=max_chunk, page_tokens=128, seed=3)
    assert (eng.op_gemm_plan(max_chunk, d, ffn)[0] == max_chunk and eng.op_gemm_plan(max_chunk, d, ffn)[2] > 1) == few_rows
    toks = si.make_tokens(1500, shape.vocab, seed=7)
    whole = _prefill_in_steps(eng, toks, [max_chunk])
    for steps in ([64], [7, 101, 120], [37], [33, 1, 90]):
        assert torch.equal(_prefill_in_steps(eng, toks, steps), whole), steps


def test_bf16_prefill_of_a_wide_model_in_steps():
    """The 8B shape: with steps of up to 128 tokens the same bits whatever the steps; with steps of up to 1024 the kernels
    go by the tokens of a step, and a short last step rounds differently (one bf16 block's flat 2e-2 of the largest value,
    tests/test_gpu_gemm_small.py)."""
    import torch
    import paper_2410_03065_amd as cake
    shape = si.SHAPES["llama3-8b-shape"].with_(n_layers=2, vocab=2048)
    toks = si.make_tokens(1200, shape.vocab, seed=11)
    eng = cake.Engine(shape, None, max_tokens=1280, max_chunk=128, page_tokens=256, seed=5)
    whole = _prefill_in_steps(eng, toks, [128])
    for steps in ([37], [101, 7, 64]):
        assert torch.equal(_prefill_in_steps(eng, toks, steps), whole), steps
    del eng
    eng = cake.Engine(shape, None, max_tokens=1280, max_chunk=1024, page_tokens=256, seed=5)
    for steps in ([1024], [512], [137, 700], [1000, 8]):
        other = _prefill_in_steps(eng, toks, steps)
        err = float((other.float() - whole.float()).abs().max() / whole.float().abs().max())
        print("steps %s: largest difference %.2e of the largest value" % (steps, err))
        assert err < 2e-2, (steps, err)
