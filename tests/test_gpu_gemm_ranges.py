"""bf16 products whose K ranges whole tiles leave to the kernel after them, or to a pass that adds them up: ragged rows,
ranges of eight slices (of 64) and of many, ranges of unequal length (persistent kernel), products beside them that stay in one
range because the pass would cost more than it saves, and a block of heads of 64."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


def _sums(eng, M, N, K):
    """max |error| / max |value| of the plain and the residual product, and whether a second run has the same bits."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N + K)
    mk = lambda r, c, std: (torch.randn(r, c, device="cuda", generator=g) * std).to(eng.tdtype)
    a, w = mk(M, K, 1.0), mk(N, K, 0.05)
    x0 = torch.randn(M, N, device="cuda", generator=g)
    want = a.double() @ w.double().t().contiguous()
    x = x0.clone()
    torch.cuda.synchronize()       # the engine's streams do not wait for torch's
    rel = lambda got, ref: float((got.double() - ref).abs().max() / ref.abs().max())
    got = eng.op_gemm(a, w)
    return rel(got, want), rel(eng.op_gemm_residual(a, w, x), x0.double() + want), torch.equal(got, eng.op_gemm(a, w))


# Float32 sums over K: 2e-6 of the largest value up to K = 256 and in proportion beyond.
@pytest.mark.parametrize("M,N,K,tile,ranges", [
    (193, 2048, 2048, (128, 128), 4), (200, 2560, 6144, (128, 128), 6), (500, 2048, 8192, (128, 128), 4), (300, 4096, 4096, (128, 128), 2),
    (512, 2048, 2048, (128, 128), 2), (257, 3072, 8192, (128, 192), 4), (320, 6144, 4096, (128, 192), 2), (193, 3072, 8192, (128, 192), 8),
    (513, 2048, 8192, (256, 256), 8), (330, 4096, 11008, (256, 256), 8),          # 172 slices in eight: 22 and 21
    (700, 4096, 11008, (256, 256), 5), (512, 5120, 13824, (256, 256), 6),
    (193, 2048, 512, (128, 64), 1), (257, 5120, 1024, (128, 64), 1)])
def test_gemm_bf16_whole_tiles_in_k_ranges(M, N, K, tile, ranges):
    import paper_2410_03065_amd as cake
    eng = cake.Engine(si.ModelShape("gemm-small", 1, 4096, 32, 8, 128, 512, 64, "bf16"), None, max_tokens=1024, max_chunk=1024, page_tokens=64)
    assert eng.op_gemm_plan(M, N, K) == tile + (ranges,)
    plain, residual, again = _sums(eng, M, N, K)
    tol = 2e-6 * max(1, K / 256)
    assert plain < tol and residual < tol and again, (plain, residual, again)


# A block of the d 2048 model with heads of 64: the rotary step, the norm and the sum after the last layer add ranges up.
# Against the generic kernels; both round the same activations to bf16, so the flat 2e-2 of a bf16 block covers both.
@pytest.mark.parametrize("begin,rows", [(0, 1), (37, 130), (37, 200), (100, 333), (64, 512), (37, 987)])
def test_block_of_heads_of_64_in_k_ranges(begin, rows):
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("hd64", 2, 2048, 32, 8, 64, 8192, 2048, "bf16", rope_theta=500000.0)
    pages = (begin + rows + 63) // 64
    eng = cake.Engine(shape, None, max_tokens=pages * 64, max_chunk=pages * 64, page_tokens=64, seed=5)
    toks = si.make_tokens(begin + rows, shape.vocab, seed=rows)
    got = []
    for path in (1, 0, 0):
        eng.clear_pool()
        eng.set_tuning(kernel_path=1)
        eng.prefill_chunk(toks, 0, begin)
        eng.set_tuning(kernel_path=path)
        eng.prefill_chunk(toks, begin, rows)
        got.append(eng.pool[1].float().clone())
        torch.cuda.synchronize()
    err = float((got[0] - got[1]).abs().max() / got[0].abs().max())
    assert err < 2e-2, err
    assert torch.equal(got[1], got[2])
