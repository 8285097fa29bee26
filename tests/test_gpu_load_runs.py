"""Unthrottled loads bring whole images, several to a copy and a kernel, into the pages; paced ones go piece by piece.  Both
leave the same bits in the range's pages and none elsewhere: ranges of fewer and more pages than the staging buffer and a
launch hold, runs whose last part is copied layer page by layer page (10 + 10 + 1 pages), a staging buffer under a raw
image, a stride larger than an image, pageable memory."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("memory", ["pinned", "stride", "pageable"])
@pytest.mark.parametrize("fmt", ["RAW", "INT8", "INT4"])
@pytest.mark.parametrize("kind,hd,n_kv,layers,pt,pages,chunk_pages", [("bf16", 64, 1, 1, 64, 71, 70), ("bf16", 64, 1, 1, 64, 21, 19), ("bf16", 128, 3, 2, 128, 9, 3),
                                                                     ("f32", 64, 2, 2, 64, 6, 4), ("bf16", 128, 2, 3, 64, 3, 1)])
def test_unthrottled_and_paced_loads_are_alike(kind, hd, n_kv, layers, pt, pages, chunk_pages, fmt, memory):
    import ctypes
    import torch
    import paper_2410_03065_amd as cake
    f = getattr(cake, "STORE_" + fmt)
    shape = si.ModelShape("load-runs", layers, 256, 2 * n_kv, n_kv, hd, 256, 64, kind)
    rng = np.random.default_rng(pages)
    eng = cake.Engine(shape, None, max_tokens=pages * pt, max_chunk=chunk_pages * pt, page_tokens=pt,
                      block_table=rng.permutation(pages).astype(np.int32))
    image = int(eng.lib.cake_store_image_bytes(ctypes.byref(cake.model_desc(shape)), pt, f))
    stride = image + (40 if memory == "stride" else 0)
    buf = torch.empty((pages, stride), dtype=torch.uint8, pin_memory=memory != "pageable")
    host = buf.numpy()
    host[:] = rng.integers(0, 120, host.shape, dtype=np.uint8)     # any bytes up to 119 are finite codes, scales and elements
    st = cake.KvStore(buf.data_ptr(), stride, pt, pages, f, cake.STORE_PINNED, -1, 0, 0)

    def load(begin, gbps):
        eng.pool.fill_(3.0)
        torch.cuda.synchronize()
        assert eng.lib.cake_load_chunk(eng.ctx, ctypes.byref(st), begin * pt, (pages - begin) * pt, ctypes.byref(eng.kv), gbps) == 0
        assert eng.lib.cake_sync_load(eng.ctx) == 0
        return eng.pool.view(torch.uint8).cpu().numpy().copy()
    for begin in (0, 1):
        np.testing.assert_array_equal(load(begin, 0.0), load(begin, 1000.0))
