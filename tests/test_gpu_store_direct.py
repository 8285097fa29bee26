"""A store written into pinned memory, with a stride that is no multiple of 16, and into pageable memory: the same bytes,
those of the pool's pages, nothing beside them, whether an image fits the staging buffer or not; and while it is written,
another context on the GPU computes."""
import ctypes
import threading
import time

import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["RAW", "INT8", "INT4"])
@pytest.mark.parametrize("kind,hd,n_kv,layers,pt,T", [("bf16", 64, 1, 1, 64, 64), ("bf16", 64, 1, 1, 64, 1344), ("bf16", 64, 3, 2, 128, 500),
                                                      ("bf16", 128, 8, 2, 256, 1300), ("f32", 64, 2, 2, 64, 300)])
@pytest.mark.parametrize("chunk_pages", [1, 8])              # a raw image is larger than the staging buffer, and fits it
def test_pinned_and_staged_stores_are_alike(fmt, kind, hd, n_kv, layers, pt, T, chunk_pages):
    import torch
    import paper_2410_03065_amd as cake
    f = getattr(cake, "STORE_" + fmt)
    shape = si.ModelShape("direct", layers, 256, 2 * n_kv, n_kv, hd, 256, 64, kind)
    n = (T + pt - 1) // pt
    bt = np.random.default_rng(T).permutation(n).astype(np.int32)
    eng = cake.Engine(shape, None, max_tokens=n * pt, max_chunk=min(n, chunk_pages) * pt, page_tokens=pt, block_table=bt)
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


@pytest.mark.parametrize("fmt", ["RAW", "INT8"])
@pytest.mark.parametrize("memory", ["pinned", "stride", "pageable"])
def test_writes_keep_off_the_slots_of_a_queued_load(fmt, memory):
    """A quantised load goes through the staging buffer while another sequence's pages are written: neither shows in the other."""
    import torch
    import paper_2410_03065_amd as cake
    f, pt, n = getattr(cake, "STORE_" + fmt), 64, 24
    shape = si.ModelShape("store-slots", 2, 256, 4, 2, 128, 256, 64, "bf16")
    eng = cake.Engine(shape, None, max_tokens=n * pt, max_chunk=4 * pt, page_tokens=pt)
    gen = torch.Generator(device="cuda").manual_seed(5)
    eng.pool.normal_(generator=gen)
    other = torch.empty_like(eng.pool).normal_(generator=gen)
    torch.cuda.synchronize()
    eng.write_store(n * pt, cake.STORE_INT8)                  # the store that is loaded
    eng.load_chunk(0, n * pt)
    loaded = eng.pool.clone()
    image = int(eng.lib.cake_store_image_bytes(ctypes.byref(cake.model_desc(shape)), pt, f))
    stride = image + (8 if memory == "stride" else 0)
    kv = cake.Kv(other.data_ptr(), eng.block_table_host.ctypes.data, eng.block_table_dev.data_ptr(), pt, n, n)
    into = torch.empty((n, stride), dtype=torch.uint8, pin_memory=memory != "pageable")

    def write():
        into.fill_(7)
        st = cake.KvStore(into.data_ptr(), stride, pt, n, f, cake.STORE_PINNED, -1, 0, 0)
        assert eng.lib.cake_write_store(eng.ctx, ctypes.byref(kv), n * pt, ctypes.byref(st)) == 0
        return into.clone()
    alone = write()
    eng.clear_pool()
    t0 = time.monotonic()
    eng.load_chunk(0, n * pt, gbps=n * eng.store_tensor.shape[1] / 0.1 / 1e9, sync=False)    # the load takes 0.1 s
    writes = 0
    while time.monotonic() - t0 < 0.08:
        assert torch.equal(write(), alone)
        writes += 1
    assert writes > 1                                         # they did not wait for the load
    eng._check(eng.lib.cake_sync_load(eng.ctx), "cake_sync_load")
    torch.cuda.synchronize()
    assert torch.equal(eng.pool, loaded)


@pytest.mark.parametrize("fmt", ["RAW", "INT8"])
def test_another_context_computes_beside_a_write(fmt):
    """A prefill of 1 ms begun while a store is being written (5 ms and more) ends before the write does."""
    import torch
    import paper_2410_03065_amd as cake
    f, T = getattr(cake, "STORE_" + fmt), 32768
    shape = si.SHAPES["llama3-8b-shape"].with_(n_layers=2, vocab=64)
    a = cake.Engine(shape.with_(n_layers=4), None, max_tokens=T, max_chunk=1024, page_tokens=256)
    overlap = ctypes.c_int32(0)
    while not overlap.value:                                  # compute streams on hardware queues of their own
        b = cake.Engine(shape, None, max_tokens=2048, max_chunk=1024, page_tokens=256)
        assert b.lib.cake_streams_overlap(a.compute_stream.cuda_stream, b.compute_stream.cuda_stream, ctypes.byref(overlap)) == 0
    toks = si.make_tokens(2048, shape.vocab, seed=1)
    a.pool.normal_()
    torch.cuda.synchronize()
    store = a.write_store(T, f).numpy()
    first, last = store[0, :256].copy(), store[-1, -256:].copy()
    b.prefill_chunk(toks, 1024, 1024)

    def write():
        assert a.lib.cake_write_store(a.ctx, ctypes.byref(a.kv), T, ctypes.byref(a.store)) == 0
    ended_beside = 0
    for _ in range(5):
        store[0, :256], store[-1, -256:] = first ^ 255, last ^ 255
        th = threading.Thread(target=write)
        th.start()
        t0 = time.monotonic()
        while not np.array_equal(store[0, :256], first) and time.monotonic() - t0 < 5:
            pass                                              # until the write is under way
        b.prefill_chunk(toks, 1024, 1024)
        ended_beside += not np.array_equal(store[-1, -256:], last)
        th.join()
        np.testing.assert_array_equal(store[-1, -256:], last)
    assert ended_beside >= 3, ended_beside
