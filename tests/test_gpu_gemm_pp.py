"""bf16 products of items of 256 rows on the kernel with eight waves in turn: one slice of K, two and three, the line between it
and the four-wave kernel (100 slices), panels of every width, ragged rows, several items to a workgroup, K ranges of unequal
length, and results that are not 16-byte aligned."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


def _engine(**tuning):
    import paper_2410_03065_amd as cake
    eng = cake.Engine(si.ModelShape("gemm-pp", 1, 4096, 32, 8, 128, 512, 64, "bf16"), None, max_tokens=1024, max_chunk=1024, page_tokens=64)
    eng.set_tuning(gemm_config=7, **tuning)
    return eng


def _operands(eng, M, N, K):
    import torch
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N + K)
    mk = lambda r, c, std: (torch.randn(r, c, device="cuda", generator=g) * std).to(eng.tdtype)
    a, w, w2, x0 = mk(M, K, 1.0), mk(N, K, 0.05), mk(N, K, 0.05), torch.randn(M, N, device="cuda", generator=g)
    torch.cuda.synchronize()       # the engine's streams do not wait for torch's
    return a, w, w2, x0


def _rel(got, want):
    return float((got.double() - want).abs().max() / want.abs().max())


# Sums: float32 over K, 2e-6 of the largest value up to K = 256 and in proportion beyond.  SwiGLU: one rounding to bf16, and 1e-6
# of the largest value for the sums in front of it.  A plain product of under 100 slices is the four-wave kernel's and a residual one
# the eight waves': the same bits into a result of zeros.  (N of 192, 320 and 448: SwiGLU only, plain ones take the generic kernel.)
@pytest.mark.parametrize("M,N,K", [
    (1, 128, 64), (128, 128, 128), (129, 192, 192), (255, 256, 64), (257, 320, 128), (256, 448, 192),
    (300, 384, 6336), (300, 384, 6400), (511, 640, 6464),                                                # 99, 100 and 101 slices
    (1024, 10240, 6400), (1000, 14336, 6464),                              # plain panels of 192 and 128, of 256 and 192 at 100 and 101
    (1000, 16640, 64), (1024, 14336, 128), (700, 33280, 192)])                                           # two rounds and more
def test_gemm_items_of_256_rows(M, N, K):
    import torch
    eng = _engine(gemm_ksplit=1)
    a, w, w2, x0 = _operands(eng, M, N, K)
    want = a.double() @ w.double().t().contiguous()
    tol = 2e-6 * max(1, K / 256)
    got = eng.op_gemm(a, w)
    assert _rel(got, want) < tol
    assert torch.equal(got, eng.op_gemm(a, w))
    assert _rel(eng.op_gemm_residual(a, w, x0.clone()), x0.double() + want) < tol
    if N % 128 == 0:
        assert torch.equal(eng.op_gemm_residual(a, w, torch.zeros_like(x0)), got)
    want = torch.nn.functional.silu(want) * (a.double() @ w2.double().t().contiguous())
    got = eng.op_gemm_swiglu(a, w, w2).double()
    assert bool(((got - want).abs() <= 2.0 ** -8 * 1.01 * want.abs() + 1e-6 * want.abs().max()).all())


@pytest.mark.parametrize("M,N,K,ranges", [(300, 512, 12800, 2), (257, 256, 12864, 2), (1024, 1024, 14336, 4)])   # 100; 101 and 100; 56
def test_gemm_k_ranges_of_items_of_256_rows(M, N, K, ranges):
    eng = _engine(gemm_ksplit=ranges)
    a, w, _, x0 = _operands(eng, M, N, K)
    want = a.double() @ w.double().t().contiguous()
    tol = 2e-6 * max(1, K / 256)
    assert _rel(eng.op_gemm(a, w), want) < tol
    assert _rel(eng.op_gemm_residual(a, w, x0.clone()), x0.double() + want) < tol


# Results that start on any element: the same bits as on 16 bytes, and nothing beside them.  The first shape goes to these
# kernels unforced, in panels of 256 and 192; the others have panels of 128 and ragged rows, two rounds of items, and (192 and
# 128 wide) the 100 slices from which on plain stores are on the eight waves too.
@pytest.mark.parametrize("M,N,K,forced", [(1024, 14336, 1024, False), (300, 384, 192, True), (700, 33280, 64, True), (1024, 10240, 6400, True)])
@pytest.mark.parametrize("offset", [1, 2, 3, 4])
def test_results_off_16_bytes(M, N, K, forced, offset):
    import torch
    eng = _engine()
    if not forced:
        eng.set_tuning()
    a, w, w2, x0 = _operands(eng, M, N, K)
    ops = eng.lib

    def swiglu(out):
        return ops.cake_op_gemm_swiglu(eng.ctx, a.data_ptr(), w.data_ptr(), w2.data_ptr(), out.data_ptr(), M, N, K)

    def residual(out):
        return ops.cake_op_gemm_residual(eng.ctx, a.data_ptr(), w.data_ptr(), out.data_ptr(), M, N, K)

    def store(out):
        return ops.cake_op_gemm(eng.ctx, a.data_ptr(), w.data_ptr(), out.data_ptr(), M, N, K)

    for op, dtype, start in ((swiglu, eng.tdtype, None), (residual, torch.float32, x0), (store, torch.float32, None)):
        got = []
        for off in (0, offset):
            buf = torch.full((M * N + 16,), 7.0, device="cuda", dtype=dtype)
            out = buf[off:off + M * N]
            if start is not None:
                out.copy_(start.flatten())
            torch.cuda.synchronize()
            assert op(out) == 0
            eng.sync()
            got.append(out.clone())
            assert bool((buf[:off] == 7.0).all()) and bool((buf[off + M * N:] == 7.0).all())
        assert torch.equal(got[0], got[1]), op.__name__
