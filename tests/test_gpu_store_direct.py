"""A store written by the kernels into pinned memory and through the staging buffer (pageable memory, a stride that is no
multiple of 16): the same bytes, those of the pool's pages, nothing beside them; more tiles than workgroups and fewer."""
import ctypes

import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["RAW", "INT8", "INT4"])
@pytest.mark.parametrize("kind,hd,n_kv,layers,pt,T", [("bf16", 64, 1, 1, 64, 64), ("bf16", 64, 3, 2, 128, 500),
                                                      ("bf16", 128, 8, 2, 256, 1300), ("f32", 64, 2, 2, 64, 300)])
def test_pinned_and_staged_stores_are_alike(fmt, kind, hd, n_kv, layers, pt, T):
    import torch
    import paper_2410_03065_amd as cake
    f = getattr(cake, "STORE_" + fmt)
    shape = si.ModelShape("direct", layers, 256, 2 * n_kv, n_kv, hd, 256, 64, kind)
    n = (T + pt - 1) // pt
    bt = np.random.default_rng(T).permutation(n).astype(np.int32)
    eng = cake.Engine(shape, None, max_tokens=n * pt, max_chunk=pt, page_tokens=pt, block_table=bt)
    eng.pool.normal_(generator=torch.Generator(device="cuda").manual_seed(T))
    torch.cuda.synchronize()
    image = int(eng.lib.cake_store_image_bytes(ctypes.byref(cake.model_desc(shape)), pt, f))

    def write(buf, address, stride):
        st = cake.KvStore(address, stride, pt, n, f, cake.STORE_PINNED, -1, 0, 0)
        assert eng.lib.cake_write_store(eng.ctx, ctypes.byref(eng.kv), T, ctypes.byref(st)) == 0
        return buf
    pinned = torch.full((n, image + 48), 7, dtype=torch.uint8, pin_memory=True)
    odd = torch.full((n, image + 8), 7, dtype=torch.uint8, pin_memory=True)
    pageable = np.full((n, image), 7, np.uint8)
    a = write(pinned, pinned.data_ptr(), image + 48).numpy()
    b = write(odd, odd.data_ptr(), image + 8).numpy()
    c = write(pageable, pageable.ctypes.data, image)
    np.testing.assert_array_equal(a[:, :image], c)
    np.testing.assert_array_equal(b[:, :image], c)
    assert (a[:, image:] == 7).all() and (b[:, image:] == 7).all()
    if fmt == "RAW":
        phys = torch.from_numpy(eng.block_table_host[:n].astype(np.int64)).cuda()
        want = eng.pool[:, phys].transpose(0, 1).contiguous().view(torch.uint8).cpu().numpy().reshape(n, image)
        np.testing.assert_array_equal(c, want)
