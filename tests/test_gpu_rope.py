"""Rotary step and page write in 16-byte pieces, through the C ABI against the oracle: every element type and head size,
whole 64-token tiles per workgroup (many tiles) and 16-token pieces (few), ranges that begin and end inside a piece."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import store as ostore
from oracle import transformer as otf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,hd", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("n_q,n_kv,tok_begin,rows", [(4, 2, 0, 1), (4, 2, 63, 2), (4, 4, 17, 46), (6, 2, 77, 211), (32, 8, 37, 731)])
def test_rope_pieces(kind, hd, n_q, n_kv, tok_begin, rows):
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("rope", 1, 256, n_q, n_kv, hd, 512, 64, kind, rope_theta=500000.0)
    pt, T = 64, tok_begin + rows
    pages = (T + pt - 1) // pt
    bt = np.random.default_rng(1).permutation(pages).astype(np.int32)
    eng = cake.Engine(shape, None, max_tokens=pages * pt, max_chunk=pages * pt, page_tokens=pt, block_table=bt)
    qkv = np.random.default_rng(rows).standard_normal((rows, (n_q + 2 * n_kv) * hd)).astype(np.float32)
    eng.pool.fill_(3.0)                       # slots of an earlier call (before tok_begin) must stay
    torch.cuda.synchronize()
    q = eng.op_rope_kv_write(torch.from_numpy(qkv).cuda(), 0, tok_begin).float().cpu().numpy()
    pos = np.arange(tok_begin, T)
    x = qkv.astype(np.float64).reshape(rows, n_q + 2 * n_kv, hd)
    want_q = otf.rope(x[:, :n_q], pos, shape.rope_theta).transpose(1, 0, 2)
    cache = otf.KVCache(1, T, n_kv, hd)
    cache.k[0, :tok_begin] = cache.v[0, :tok_begin] = 3.0
    cache.k[0, tok_begin:] = otf.rope(x[:, n_q:n_q + n_kv], pos, shape.rope_theta)
    cache.v[0, tok_begin:] = otf.round_storage(x[:, n_q + n_kv:], kind)
    want = ostore.decode_words(ostore.pack_store(cache, pt, "f32"), "f32")   # K unrounded; zeros past the range
    got = eng.pool_images(T)
    # against the unrounded value: one rounding to bf16 (2^-8 of it), two products and a sum in float32 (1 % of that)
    tol = 2e-6 if kind == "f32" else 2.0 ** -8 * 1.01
    assert np.all(np.abs(q - want_q) <= tol * np.abs(want_q) + 1e-6)
    assert np.all(np.abs(got - want) <= tol * np.abs(want) + 1e-6)
    np.testing.assert_array_equal(got[:, :, 1], want[:, :, 1])            # V is a copy


@pytest.mark.parametrize("kind,hd", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("odd", ["pool", "q", "qkv"])
def test_rope_of_pointers_off_16_bytes(kind, hd, odd):
    """One element off 16 bytes the kernel of single elements runs: the same bits."""
    import ctypes
    import torch
    import paper_2410_03065_amd as cake
    n_q, n_kv, pt, tok_begin, rows = 6, 2, 64, 77, 211
    shape = si.ModelShape("rope-odd", 1, 256, n_q, n_kv, hd, 512, 64, kind)
    pages = (tok_begin + rows + pt - 1) // pt
    bt = np.random.default_rng(2).permutation(pages).astype(np.int32)
    eng = cake.Engine(shape, None, max_tokens=pages * pt, max_chunk=pages * pt, page_tokens=pt, block_table=bt)
    qkv = torch.from_numpy(np.random.default_rng(rows).standard_normal((rows, (n_q + 2 * n_kv) * hd)).astype(np.float32)).cuda()

    def run(offset):
        def place(n, dtype, here):
            t = torch.full((n + 4,), 3.0, dtype=dtype, device="cuda")
            return t[1:n + 1] if here else t[:n]
        pool = place(eng.pool.numel(), eng.tdtype, offset == "pool")
        q = place(n_q * rows * hd, eng.tdtype, offset == "q")
        x = place(qkv.numel(), torch.float32, offset == "qkv")
        x.copy_(qkv.flatten())
        kv = cake.Kv(pool.data_ptr(), eng.block_table_host.ctypes.data, eng.block_table_dev.data_ptr(), pt, pages, pages)
        torch.cuda.synchronize()
        assert eng.lib.cake_op_rope_kv_write(eng.ctx, x.data_ptr(), q.data_ptr(), 0, tok_begin, rows, ctypes.byref(kv)) == 0
        eng.sync()
        return q.cpu(), pool.cpu()
    for got, want in zip(run(odd), run(None)):
        assert torch.equal(got, want)
