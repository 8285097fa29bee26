"""float32 prefill whose QKV and gate/up products norm their input themselves, on every tile (16, 32 and 64 square with K divided
among the waves, 128 square), ragged rows and a K that is no multiple of 32, against the plain kernels with the norm apart."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

NARROW = si.ModelShape("f32-narrow", 2, 256, 4, 2, 64, 688, 512, "f32")
ODD = si.ModelShape("f32-odd", 2, 200, 3, 1, 64, 296, 512, "f32")
WIDE = si.ModelShape("f32-wide", 2, 1536, 24, 12, 64, 4096, 512, "f32")


# Both sides sum float32 products: 2e-6 of the largest value up to K = 256 and in proportion beyond for each of the block's
# products, of which three stand in a row between the embedding and the second layer's K and V.
@pytest.mark.parametrize("shape,begin,rows", [
    (NARROW, 0, 1), (NARROW, 5, 15), (NARROW, 0, 33), (NARROW, 130, 256), (NARROW, 0, 1000),
    (ODD, 3, 70), (WIDE, 0, 100), (WIDE, 0, 500), (WIDE, 0, 1024)], ids=lambda v: v.name if hasattr(v, "name") else str(v))
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
