"""One-token attention over every size of head group: one and two columns of sixteen heads, eight and four waves, and
prompts that end inside a 32-key tile, a page, a key range; the vector-ALU kernel on the same cache beside it."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import transformer as otf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q,n_kv,T", [(1, 1, 1), (3, 3, 33), (12, 1, 257), (13, 1, 64), (16, 1, 1000), (34, 2, 131),
                                        (32, 1, 2049), (10, 2, 30011)])
def test_decode_attention_head_groups(n_q, n_kv, T):
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("groups", 1, 256, n_q, n_kv, 128, 256, 64, "bf16")
    pages = (T + 63) // 64
    bt = np.random.default_rng(T).permutation(pages).astype(np.int32)
    eng = cake.Engine(shape, None, max_tokens=pages * 64, max_chunk=64, page_tokens=64, block_table=bt, with_head=True)
    eng.pool.normal_(generator=torch.Generator(device="cuda").manual_seed(T))
    q = np.random.default_rng(n_q).standard_normal((n_q, 128)).astype(np.float32) * 2
    Q = torch.from_numpy(q).cuda()
    torch.cuda.synchronize()
    got = eng.op_decode_attention(Q, 0, T).cpu().numpy()
    half = n_kv * 64 * 128
    pool = eng.pool[0, torch.from_numpy(bt.astype(np.int64)).cuda()].double().cpu().numpy()
    k = pool[:, :half].reshape(pages, n_kv, 64, 128).transpose(0, 2, 1, 3).reshape(-1, n_kv, 128)[:T]
    v = pool[:, half:].reshape(pages, n_kv, 128, 64).transpose(0, 3, 1, 2).reshape(-1, n_kv, 128)[:T]
    want = otf.attention(q.astype(np.float64)[None], k, v, np.array([T - 1]), np.arange(T))[0]
    # q and the probabilities are rounded to bf16 (2^-9 each, the first in the exponent): as the other bound of this kernel
    assert np.abs(got - want).max() < 1.2e-2 * np.abs(want).max()
    eng.set_tuning(kernel_path=1)
    if n_q // n_kv in (1, 2, 4, 8):
        ref = eng.op_decode_attention(Q, 0, T).cpu().numpy()
        assert np.abs(ref - want).max() < 2e-5 * np.abs(want).max()
