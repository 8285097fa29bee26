"""What a prefill begins with: token ids in the launch's arguments (up to 512 rows) and in device memory, rows whose first norm is
in that launch (multiples of 1024) and others, in pieces of 16 bytes and off them, float32 and bf16, positions away from 0, a
captured step."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

SHAPES = [si.ModelShape("begin-%s-%d" % (dt, d), 1, d, d // 64, 1, 64, 256, 1000, dt) for dt, d in (("f32", 256), ("f32", 1024), ("bf16", 448), ("bf16", 2048))]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
@pytest.mark.parametrize("rows", [1, 63, 511, 512, 513])
def test_ids_in_arguments_and_in_memory(shape, rows):
    """Both routes give the same bits: one call for the rows, and the same rows as the only chunk of a computed prompt."""
    import paper_2410_03065_amd as cake
    import torch
    eng = cake.Engine(shape, None, max_tokens=640, max_chunk=640, page_tokens=64, seed=2)
    toks = si.make_tokens(rows, shape.vocab, seed=rows)
    eng.prefill_chunk(toks, 0, rows)
    want = eng.pool.clone()
    torch.cuda.synchronize()
    eng.clear_pool()
    eng.bidirectional_prefill(toks, 640, 0.0, mode="compute_only")
    assert torch.equal(eng.pool, want) and float(want.abs().max()) > 0


@pytest.mark.parametrize("d,rows", [(72, 3), (2568, 150), (2048, 150), (9216, 20)])
def test_embedding_rows_on_and_off_16_bytes(d, rows):
    """bf16 rows of 9, 321 (two trips, the second short), 256 and 1152 pieces; the table moved by one element and by 16 bytes."""
    import ctypes
    import paper_2410_03065_amd as cake
    import torch
    shape = si.ModelShape("begin-off", 1, d, 2, 1, 64, 256, 1000, "bf16")
    eng = cake.Engine(shape, None, max_tokens=192, max_chunk=192, page_tokens=64, seed=2)
    toks, want = si.make_tokens(rows, shape.vocab, seed=rows), None
    for offset in (0, 1, 8):
        table = torch.zeros(shape.vocab * d + 16, device="cuda", dtype=eng.tdtype)
        table[offset:offset + shape.vocab * d] = eng.embed.flatten()
        torch.cuda.synchronize()
        eng.lib.cake_destroy(eng.ctx)
        eng._weights.embed = table.data_ptr() + 2 * offset
        desc = cake.model_desc(shape)
        assert eng.lib.cake_create(ctypes.byref(eng.ctx), ctypes.byref(desc), ctypes.byref(eng._weights), 192, 192,
                                   eng.compute_stream.cuda_stream, eng.copy_stream.cuda_stream) == 0
        eng.clear_pool()
        eng.prefill_chunk(toks, 0, rows)
        want = eng.pool.clone() if want is None else want
        assert torch.equal(eng.pool, want) and float(want.abs().max()) > 0


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_first_norm_and_rotary_table(shape):
    """Against the plain kernels and the oracle's embedding of the same tokens: K is the rotated product of the normed rows."""
    import numpy as np
    import paper_2410_03065_amd as cake
    import torch
    begin, rows = 70, 150
    eng = cake.Engine(shape, None, max_tokens=256, max_chunk=256, page_tokens=64, seed=2)
    t = eng.layer_tensors[0]
    t["attn_norm"].mul_(1 + 0.3 * torch.randn(shape.d_model, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)))
    torch.cuda.synchronize()
    toks = si.make_tokens(begin + rows, shape.vocab, seed=7)
    eng.prefill_chunk(toks, begin, rows)
    x = eng.embed[torch.from_numpy(toks[begin:].astype(np.int64)).cuda()].double()
    h = x * torch.rsqrt((x * x).mean(dim=1, keepdim=True) + shape.rms_eps) * t["attn_norm"].double()
    hd, hq = 64, shape.n_q * 64
    k = (h @ t["wqkv"][hq:hq + hd].double().t().contiguous())
    ang = torch.arange(begin, begin + rows, device="cuda", dtype=torch.float64)[:, None] * shape.rope_theta ** (-torch.arange(hd // 2, device="cuda", dtype=torch.float64) * 2 / hd)
    c, s = ang.cos(), ang.sin()
    want = torch.stack([k[:, 0::2] * c - k[:, 1::2] * s, k[:, 0::2] * s + k[:, 1::2] * c], dim=-1).flatten(1)
    pages = eng.pool[0][torch.from_numpy(eng.block_table_host.astype(np.int64)).cuda()]
    got = pages[:, :64 * hd].reshape(-1, hd)[begin:begin + rows].double()
    # float32: sums over d_model and a float32 table; bf16: one rounding of h and one of K, against the largest value
    tol = 1e-5 if shape.dtype == "f32" else 2.0 ** -7
    assert float((got - want).abs().max() / want.abs().max()) < tol


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_bytes_of_the_first_launch(shape):
    """The profile counts the normed rows in the launch that writes them: the begin of a bf16 prefill whose rows are whole pieces
    of 1024, the norm's own launch elsewhere, no launch where the product norms its input (float32)."""
    import paper_2410_03065_amd as cake
    eng = cake.Engine(shape, None, max_tokens=128, max_chunk=128, page_tokens=64, seed=2)
    eng.profile_enable(True)
    rows, d, e = 100, shape.d_model, shape.elem_bytes
    eng.prefill_chunk(si.make_tokens(rows, shape.vocab, seed=1), 0, rows)
    got = eng.profile_read()
    inside = shape.dtype == "bf16" and d % 1024 == 0
    assert got["embed"]["bytes"] == rows * d * (e + 4 + (e if inside else 0))
    assert got["rmsnorm"]["bytes"] == rows * d * (4 + e) * (0 if shape.dtype == "f32" else 1 if inside else 2)


def test_captured_step_reads_its_ids_anew():
    """In a captured stream the ids stay a copy: a replay takes what the caller's array then holds."""
    import paper_2410_03065_amd as cake
    import torch
    shape = SHAPES[3]
    eng = cake.Engine(shape, None, max_tokens=256, max_chunk=256, page_tokens=64, seed=2)
    ids, other = si.make_tokens(100, shape.vocab, seed=1), si.make_tokens(100, shape.vocab, seed=9)
    want = []
    for t in (ids, other):
        eng.clear_pool()
        eng.prefill_chunk(t, 0, 100)
        want.append(eng.pool.clone())
        torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    held = ids.copy()
    with torch.cuda.graph(graph, stream=eng.compute_stream):
        eng.prefill_chunk(held, 0, 100, sync=False)
    held = eng._keep     # the array that the call was given
    for t, w in ((ids, want[0]), (other, want[1]), (ids, want[0])):
        held[:] = t
        eng.clear_pool()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(eng.pool, w)
        assert float(torch.ones(64, device="cuda").sum()) == 64     # eager work between the replays
