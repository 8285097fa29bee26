"""GEMM kernels for few rows and for float32 models, through the C ABI's op calls against a float64 product: every
tile of the dispatch, with rows, columns and K that end inside one."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


def _products(kind, M, N, K):
    """max |error| / max |value| of the three epilogues (SwiGLU: largest error over 2^-8 resp. 2^-17 of each value)."""
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("gemm-small", 1, 256, 4, 4, 64, 512, 64, kind)
    eng = cake.Engine(shape, None, max_tokens=1024, max_chunk=1024, page_tokens=64)
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N + K)
    mk = lambda r, c, std: (torch.randn(r, c, device="cuda", generator=g) * std).to(eng.tdtype)
    a, w, w2 = mk(M, K, 1.0), mk(N, K, 0.05), mk(N, K, 0.05)
    x0 = torch.randn(M, N, device="cuda", generator=g)
    want = a.double() @ w.double().t().contiguous()
    up = a.double() @ w2.double().t().contiguous()
    x = x0.clone()
    torch.cuda.synchronize()       # the engine's streams do not wait for torch's
    rel = lambda got, ref: float((got.double() - ref).abs().max() / ref.abs().max())
    plain = rel(eng.op_gemm(a, w), want)
    again = torch.equal(eng.op_gemm(a, w), eng.op_gemm(a, w))
    residual = rel(eng.op_gemm_residual(a, w, x), x0.double() + want)
    ref = torch.nn.functional.silu(want) * up
    got = eng.op_gemm_swiglu(a, w, w2).double()
    bound = (2.0 ** -17 if kind == "f32" else 2.0 ** -8 * 1.01) * ref.abs() + 1e-6 * ref.abs().max()
    return plain, residual, float(((got - ref).abs() / bound).max()), again


# float32 sums over K: 2e-6 of the largest value up to K = 256 and in proportion beyond (a bound of K * 2^-24 on a
# sum's relative error, taken at the spread of these operands)
@pytest.mark.parametrize("M,N,K", [
    (1, 5, 8), (17, 15, 40), (256, 256, 256), (33, 1376, 72),         # 16 x 16 tiles, K in fewer and more pieces than waves
    (256, 768, 256), (500, 321, 104),                                 # 32 x 32
    (1000, 1300, 136), (1024, 3072, 96),                              # 64 x 64 and 128 x 128
])
def test_gemm_f32(M, N, K):
    plain, residual, swiglu, again = _products("f32", M, N, K)
    tol = 2e-6 * max(1, K / 256)
    assert plain < tol and residual < tol and swiglu < 1.0 and again, (plain, residual, swiglu, again)


# The tile is chosen from the rows (16 x 16 to 128 x 128), the order of a sum is not: a row has the same bits beside any
# others.
@pytest.mark.parametrize("M,N,K", [(1024, 3072, 328), (1024, 1376, 1000), (300, 688, 40), (897, 6400, 128)])
def test_gemm_f32_rows_do_not_depend_on_the_rows_beside_them(M, N, K):
    import torch
    import paper_2410_03065_amd as cake
    eng = cake.Engine(si.ModelShape("gemm-small", 1, 256, 4, 4, 64, 512, 64, "f32"), None, max_tokens=64, max_chunk=64, page_tokens=64)
    g = torch.Generator(device="cuda").manual_seed(N)
    mk = lambda r, c, std: torch.randn(r, c, device="cuda", generator=g) * std
    a, w, w2, x0 = mk(M, K, 1.0), mk(N, K, 0.05), mk(N, K, 0.05), mk(M, N, 1.0)

    def products(lo, n):
        rows, x = a[lo:lo + n].contiguous(), x0[lo:lo + n].clone()
        torch.cuda.synchronize()
        return eng.op_gemm(rows, w), eng.op_gemm_residual(rows, w, x), eng.op_gemm_swiglu(rows, w, w2)
    whole = products(0, M)
    for lo, n in [(0, 1), (M - 1, 1), (5, 37), (64, 101), (100, 200), (0, min(M, 512))]:
        for name, got, want in zip(("store", "residual", "swiglu"), products(lo, n), whole):
            assert torch.equal(got, want[lo:lo + n]), (name, lo, n)


# A block whose products leave K ranges to the kernel after them (few rows: one tile of all rows; many: the persistent
# kernel), against the generic kernels on the same weights.  Both round the same activations to bf16, so what differs is
# float32 summation order, which flips single roundings: the flat 2e-2 of a bf16 block covers both against the exact value.
@pytest.mark.parametrize("base,rows", [("llama3-8b-shape", r) for r in (1, 31, 33, 100, 137, 192, 193, 700, 1024)] +
                         [("llama2-7b-shape", 64), ("llama2-7b-shape", 1000), ("longalpaca-13b-shape", 512)])
def test_block_with_products_left_in_k_ranges(base, rows):
    import torch
    import paper_2410_03065_amd as cake
    shape = si.SHAPES[base].with_(n_layers=2, vocab=2048)
    begin = 37
    T = begin + rows
    pages = (T + 63) // 64
    eng = cake.Engine(shape, None, max_tokens=pages * 64, max_chunk=min(1024, pages * 64), page_tokens=64, seed=5)
    toks = si.make_tokens(T, shape.vocab, seed=rows)
    got = []
    for path in (1, 0):
        eng.clear_pool()
        eng.set_tuning(kernel_path=1)
        eng.prefill_chunk(toks, 0, begin)
        eng.set_tuning(kernel_path=path)
        eng.prefill_chunk(toks, begin, rows)
        got.append(eng.pool[1].float().clone())
        torch.cuda.synchronize()
    err = float((got[0] - got[1]).abs().max() / got[0].abs().max())
    print("%s rows %d: largest difference %.2e of the largest value" % (base, rows, err))
    assert err < 2e-2, err
    eng.set_tuning(kernel_path=0)
    eng.prefill_chunk(toks, begin, rows)                       # the same bits again
    assert torch.equal(eng.pool[1].float(), got[1])


# Narrow bf16 products of few rows, on the ordinary tiles: float32 sums over K as above; SwiGLU rounds once to bf16 (2^-8
# of a value)
@pytest.mark.parametrize("M,N,K", [(129, 128, 64), (137, 384, 512), (192, 640, 4096), (33, 256, 192), (160, 64, 128)])
def test_gemm_bf16_few_rows(M, N, K):
    plain, residual, swiglu, again = _products("bf16", M, N, K)
    tol = 2e-6 * max(1, K / 256)
    assert plain < tol and residual < tol and swiglu < 1.0 and again, (plain, residual, swiglu, again)


# Plain and residual products of up to 192 rows that are taken in K ranges by one tile of all rows and added up by a pass
# of its own: every tile height, ranges of one slice (64) and of many.
@pytest.mark.parametrize("M,N,K,ranges", [
    (1, 2048, 512, 8), (1, 4096, 4096, 8), (33, 4096, 4096, 8), (64, 2048, 8192, 8), (96, 2176, 1024, 4), (128, 4096, 4096, 8),
    (129, 4096, 4096, 8), (137, 6144, 4096, 4), (192, 4096, 4096, 8)])
def test_gemm_bf16_few_rows_in_k_ranges(M, N, K, ranges):
    import paper_2410_03065_amd as cake
    eng = cake.Engine(si.ModelShape("gemm-small", 1, 256, 4, 4, 64, 512, 64, "bf16"), None, max_tokens=1024, max_chunk=1024, page_tokens=64)
    for residual in (False, True):
        assert eng.op_gemm_plan(M, N, K, residual) == ((M + 31) // 32 * 32, 128, ranges)
    plain, residual, swiglu, again = _products("bf16", M, N, K)
    tol = 2e-6 * max(1, K / 256)
    assert plain < tol and residual < tol and swiglu < 1.0 and again, (plain, residual, swiglu, again)


# Gate/up of 129 to 192 rows in one tile of 192 (wide feed-forward layers only: 9216 columns and more here), and the rows
# on both sides of that; K from one slice of 64 to more than its ring holds.
@pytest.mark.parametrize("M,N,K", [(128, 9216, 64), (129, 9216, 64), (137, 11008, 320), (160, 10240, 128), (192, 9216, 192), (193, 9216, 192),
                                   (150, 14336, 1024)])
def test_gemm_swiglu_in_one_tile_of_192_rows(M, N, K):
    _, _, swiglu, again = _products("bf16", M, N, K)
    assert swiglu < 1.0 and again, (swiglu, again)
