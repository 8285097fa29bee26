"""The first-token step's products at sizes where a row ends inside a piece, a set of pieces or a group of rows, against
the oracle's logits, and the arg max among equal logits."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import store as ostore
from oracle import transformer as otf

pytestmark = pytest.mark.gpu


# float32 sums: 2e-5 of the largest logit (d up to 2056 terms); bf16 pages: the one-token attention rounds its query and
# probabilities to bf16 (2^-9 each) in a residual stream that it only adds to: 1e-2
@pytest.mark.parametrize("kind,d,n_q,n_kv,hd,ffn,vocab,T", [
    ("f32", 1000, 4, 2, 64, 2760, 1003, 70),
    ("f32", 2056, 4, 4, 64, 520, 16387, 5),       # normed input staged, a row ends inside a piece; four rows per wave
    ("bf16", 1000, 4, 2, 128, 2760, 517, 130),
    ("bf16", 2056, 8, 2, 128, 1032, 16387, 33),
    ("bf16", 4096, 4, 4, 128, 264, 301, 64),      # whole sets only
])
def test_first_token_products(kind, d, n_q, n_kv, hd, ffn, vocab, T):
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("first-token", 2, d, n_q, n_kv, hd, ffn, vocab, kind, rope_theta=500000.0)
    w = si.make_weights(shape, seed=3, gain_jitter=0.2, with_head=True)
    toks = si.make_tokens(T, vocab, seed=4)
    ref = otf.prefill_chunked(w, shape, toks, 64, kv_dtype=kind)
    eng = cake.Engine(shape, w, max_tokens=256, max_chunk=256, page_tokens=64)
    images = ostore.pack_store(ref, 64, kind)
    eng.set_store(images)
    eng.load_chunk(0, T)
    tok, _, logits = eng.first_token(toks, want_logits=True)
    want = otf.first_token_logits(w, shape, toks, ref)
    scale = np.abs(want).max()
    err = float(np.abs(logits - want).max() / scale)
    print("first token %s d=%d: largest error %.2e of the largest logit" % (kind, d, err))
    assert err < (2e-5 if kind == "f32" else 1e-2), err
    assert tok == int(np.argmax(logits))          # the lowest index of its own largest logit
    assert eng.first_token(toks)[0] == tok        # without the logits, from the same state


def test_first_of_equal_logits():
    """Every row of the head the same: all logits equal, the first index wins over all workgroups' pieces."""
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("first-token-ties", 1, 256, 4, 4, 64, 256, 40000, "f32")
    eng = cake.Engine(shape, None, max_tokens=64, max_chunk=64, page_tokens=64, with_head=True)
    toks = si.make_tokens(10, shape.vocab, seed=1)
    eng.prefill_chunk(toks, 0, 10)
    eng.lm_head[:] = eng.lm_head[0].clone()
    torch.cuda.synchronize()
    assert eng.first_token(toks)[0] == 0
    eng.lm_head[:31000] *= 0.5
    eng.lm_head[:] = eng.lm_head * torch.sign(torch.tensor(float(eng.first_token(toks, want_logits=True)[2][39999])))
    torch.cuda.synchronize()
    assert eng.first_token(toks)[0] == 31000


@pytest.mark.parametrize("kind,d,hd", [("f32", 1000, 64), ("f32", 2048, 64), ("bf16", 1000, 128), ("bf16", 4096, 128)])
def test_norm_gains_aligned_to_their_elements_only(kind, d, hd):
    """Gains at addresses 4, 8 and 12 past a multiple of 16 give the same logits as aligned ones."""
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("first-token-gains", 2, d, 4, 2, hd, 512, 301, kind)

    class Shifted(cake.Engine):
        def _build_weights(self, weights, seed):
            super()._build_weights(weights, seed)
            g = torch.Generator(device=self.dev).manual_seed(9)

            def moved(by):
                t = torch.zeros(d + 4, device=self.dev)[by:by + d]
                t.copy_(torch.rand(d, device=self.dev, generator=g) + 0.5)
                self._tensors.append(t)
                return t.data_ptr()
            for l in range(shape.n_layers):
                self._layer_arr[l].attn_norm, self._layer_arr[l].ffn_norm = moved(self.shift), moved(self.shift)
            self._weights.final_norm = moved(self.shift)
    logits = []
    for by in range(4):
        eng = type("E", (Shifted,), {"shift": by})(shape, None, max_tokens=64, max_chunk=64, page_tokens=64, seed=2, with_head=True)
        eng.pool.normal_(generator=torch.Generator(device="cuda").manual_seed(1))
        torch.cuda.synchronize()
        logits.append(eng.first_token(si.make_tokens(50, shape.vocab, seed=1), want_logits=True)[2].copy())
    for other in logits[1:]:
        assert np.array_equal(other, logits[0])
