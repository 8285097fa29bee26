"""float32 prefill whose QKV and gate/up products norm their input themselves, on every tile that does (16, 32 and 64 square), and
contexts with a norm apart in front of one or both (products of 3.5 GFLOP, 128 square tiles), ragged rows and columns and a K
that is no multiple of 32: against the plain kernels, in different steps, with rows that have no finite norm."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

NARROW = si.ModelShape("f32-narrow", 2, 256, 4, 2, 64, 688, 512, "f32")
ODD = si.ModelShape("f32-odd", 2, 200, 3, 1, 64, 296, 512, "f32")
MID = si.ModelShape("f32-mid", 2, 1024, 16, 4, 64, 2816, 512, "f32")
WIDE = si.ModelShape("f32-wide", 2, 1536, 24, 12, 64, 4096, 512, "f32")


# Both sides sum float32 products: 2e-6 of the largest value up to K = 256 and in proportion beyond for each of the block's
# products, of which three stand in a row between the embedding and the second layer's K and V.
@pytest.mark.parametrize("shape,begin,rows", [
    (NARROW, 0, 1), (NARROW, 5, 15), (NARROW, 0, 33), (NARROW, 130, 256), (NARROW, 0, 1000),
    (ODD, 3, 70), (MID, 0, 1000), (WIDE, 0, 100), (WIDE, 0, 500), (WIDE, 0, 1024)], ids=lambda v: v.name if hasattr(v, "name") else str(v))
def test_f32_products_norm_their_input(shape, begin, rows):
    import paper_2410_03065_amd as cake
    import torch
    pages = (begin + rows + 63) // 64
    eng = cake.Engine(shape, None, max_tokens=pages * 64, max_chunk=pages * 64, page_tokens=64, seed=3)
    for l, t in enumerate(eng.layer_tensors):      # gains that are not 1
        g = torch.Generator(device="cuda").manual_seed(l)
        t["attn_norm"].mul_(1 + 0.3 * torch.randn(shape.d_model, device="cuda", generator=g))
        t["ffn_norm"].mul_(1 + 0.3 * torch.randn(shape.d_model, device="cuda", generator=g))
    torch.cuda.synchronize()
    toks = si.make_tokens(begin + rows, shape.vocab, seed=rows)
    got = []
    for path in (1, 0):
        eng.clear_pool()
        eng.set_tuning(kernel_path=1)
        eng.prefill_chunk(toks, 0, begin)
        eng.set_tuning(kernel_path=path)
        eng.prefill_chunk(toks, begin, rows)
        got.append(eng.pool[1].clone())
        torch.cuda.synchronize()
    err = float((got[0] - got[1]).abs().max() / got[0].abs().max())
    assert err < 3 * 2e-6 * max(1, shape.d_model / 256), err


# Inside on tiles of 16, 32 and 64 in turn; apart before QKV only; apart before both, with 128 square tiles, ragged in all three sizes.
@pytest.mark.parametrize("d,n_q,n_kv,ffn", [(1024, 16, 4, 2816), (1536, 24, 12, 1376), (1544, 24, 12, 4104)])
def test_f32_prefill_of_wide_models_does_not_depend_on_its_steps(d, n_q, n_kv, ffn):
    import paper_2410_03065_amd as cake
    import torch
    shape = si.ModelShape("f32-wide-steps", 2, d, n_q, n_kv, 64, ffn, 128, "f32")
    eng = cake.Engine(shape, None, max_tokens=1024, max_chunk=1024, page_tokens=128, seed=3)
    toks = si.make_tokens(1000, shape.vocab, seed=7)
    got = []
    for steps in ([1000], [500], [37, 101, 300], [256]):
        eng.clear_pool()
        at, i = 0, 0
        while at < len(toks):
            n = min(steps[i % len(steps)], len(toks) - at)
            eng.prefill_chunk(toks, at, n)
            at, i = at + n, i + 1
        torch.cuda.synchronize()
        got.append(eng.pool.clone())
        assert torch.equal(got[0], got[-1]), steps


@pytest.mark.parametrize("shape", [NARROW, MID], ids=lambda s: s.name)
def test_rows_without_a_finite_norm(shape):
    """An infinity, a NaN, zeros and squares beyond float32 in a row: NaN and zero where the norm apart has them."""
    import paper_2410_03065_amd as cake
    import numpy as np
    import torch
    eng = cake.Engine(shape, None, max_tokens=256, max_chunk=256, page_tokens=64, seed=3)
    eng.embed[5, 7], eng.embed[6, 9], eng.embed[8, 3], eng.embed[9, 11] = float("inf"), float("nan"), 1e25, -float("inf")
    eng.embed[7] = 0
    torch.cuda.synchronize()
    mixed = si.make_tokens(200, shape.vocab, seed=4)
    mixed[[0, 17, 90, 130, 199]] = (5, 6, 7, 8, 9)
    # every layer of a token alone; the first layer (of the others only the attention differs) of a prompt with all of them
    for toks, layers in [(np.full(n, t, np.int32), 2) for t in (5, 6, 7, 8, 9) for n in (1, 70)] + [(mixed, 1)]:
        got = []
        for path in (1, 0):
            eng.clear_pool()
            eng.set_tuning(kernel_path=path)
            eng.prefill_chunk(toks, 0, len(toks))
            got.append(eng.pool[:layers].clone())
            torch.cuda.synchronize()
        assert torch.equal(got[0].isnan(), got[1].isnan())
        a, b = (g.nan_to_num(0.0) for g in got)
        # the sums' bound above; a prompt of zeros and NaN is the same
        assert float((a - b).abs().max()) <= 2 * 2e-6 * max(1, shape.d_model / 256) * float(a.abs().max())
