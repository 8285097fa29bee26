"""The store's quantising and expanding kernels bit for bit against the oracle: both head sizes and code widths, ragged
prompts, more pages than the staging buffer holds, a page stride larger than an image, rows of zeros."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import store as ostore
from oracle import transformer as otf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("kind,hd,n_kv,T,pt", [("bf16", 64, 2, 700, 64), ("bf16", 128, 3, 1000, 128), ("bf16", 128, 1, 320, 320), ("f32", 64, 2, 300, 64)])
def test_quantised_store_round_trip(bits, kind, hd, n_kv, T, pt):
    import paper_2410_03065_amd as cake
    fmt = cake.STORE_INT8 if bits == 8 else cake.STORE_INT4
    pack, unpack = (ostore.pack_store_int8, ostore.unpack_store_int8) if bits == 8 else (ostore.pack_store_int4, ostore.unpack_store_int4)
    shape = si.ModelShape("store-kernels", 2, 256, 2 * n_kv, n_kv, hd, 256, 64, kind)
    n = (T + pt - 1) // pt
    bt = np.random.default_rng(2).permutation(n).astype(np.int32)
    eng = cake.Engine(shape, None, max_tokens=n * pt, max_chunk=min(2 * pt, n * pt), page_tokens=pt, block_table=bt)
    rng = np.random.default_rng(T)
    cache = otf.KVCache(2, T, n_kv, hd)
    cache.k[:] = otf.round_storage(rng.standard_normal(cache.k.shape) * 4, kind)
    cache.v[:] = otf.round_storage(rng.standard_normal(cache.v.shape) * np.exp(rng.standard_normal((2, T, n_kv, 1))), kind)
    cache.v[0, 5] = 0.0
    eng.set_store(ostore.pack_store(cache, pt, kind))
    eng.load_chunk(0, T)
    images = pack(cache, pt)
    t = eng.write_store(T, fmt).numpy().reshape(images.shape)
    np.testing.assert_array_equal(t, images)
    eng.clear_pool()
    eng.load_chunk(0, T)                                          # from the quantised store just written
    want = ostore.pack_store(unpack(images, T, n_kv, hd, pt, kind), pt, kind)
    np.testing.assert_array_equal(eng.pool_raw(T).view(want.dtype), want)


def test_quantised_store_with_a_larger_stride():
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("store-stride", 1, 256, 2, 2, 128, 256, 64, "bf16")
    eng = cake.Engine(shape, None, max_tokens=512, max_chunk=256, page_tokens=128)
    eng.pool.normal_()
    torch.cuda.synchronize()
    dense = eng.write_store(512, cake.STORE_INT8).numpy().copy()
    wide = torch.zeros((4, dense.shape[1] + 96), dtype=torch.uint8, pin_memory=True)
    st = cake.KvStore(wide.data_ptr(), wide.shape[1], 128, 4, cake.STORE_INT8, cake.STORE_PINNED, -1, 0, 0)
    import ctypes
    assert eng.lib.cake_write_store(eng.ctx, ctypes.byref(eng.kv), 512, ctypes.byref(st)) == 0
    np.testing.assert_array_equal(wide.numpy()[:, :dense.shape[1]], dense)
    assert not wide.numpy()[:, dense.shape[1]:].any()


@pytest.mark.parametrize("bits", [8, 4])
def test_write_store_beside_a_queued_load(bits):
    """Quantised pages are loaded through the context's staging slots while another sequence's pages are written to a
    store from the same context: both come out as each does alone."""
    import ctypes
    import time
    import torch
    import paper_2410_03065_amd as cake
    fmt = cake.STORE_INT8 if bits == 8 else cake.STORE_INT4
    shape = si.ModelShape("store-beside", 2, 256, 4, 2, 128, 256, 64, "bf16")
    pt, n = 64, 24
    eng = cake.Engine(shape, None, max_tokens=n * pt, max_chunk=4 * pt, page_tokens=pt)      # four 8-bit slots
    g = torch.Generator(device="cuda").manual_seed(5)
    eng.pool.normal_(generator=g)
    other = torch.empty_like(eng.pool).normal_(generator=g)
    torch.cuda.synchronize()
    eng.write_store(n * pt, fmt)                                   # the store that is loaded
    eng.clear_pool()
    eng.load_chunk(0, n * pt)
    loaded = eng.pool.clone()
    kv = cake.Kv(other.data_ptr(), eng.block_table_host.ctypes.data, eng.block_table_dev.data_ptr(), pt, n, n)
    image = eng.store_tensor.shape[1]

    def write(into):
        st = cake.KvStore(into.data_ptr(), image, pt, n, fmt, cake.STORE_PINNED, -1, 0, 0)
        assert eng.lib.cake_write_store(eng.ctx, ctypes.byref(kv), n * pt, ctypes.byref(st)) == 0
    alone = torch.zeros((n, image), dtype=torch.uint8, pin_memory=True)
    write(alone)
    eng.clear_pool()
    beside = torch.zeros((n, image), dtype=torch.uint8, pin_memory=True)
    gbps = n * image / 0.1 / 1e9                                   # the load takes 0.1 s
    t0 = time.monotonic()
    eng.load_chunk(0, n * pt, gbps=gbps, sync=False)
    writes = 0
    while time.monotonic() - t0 < 0.08:
        beside.zero_()
        write(beside)
        assert torch.equal(beside, alone)
        writes += 1
    assert writes > 1                                              # they did not wait for the load
    eng._check(eng.lib.cake_sync_load(eng.ctx), "cake_sync_load")
    torch.cuda.synchronize()
    assert torch.equal(eng.pool, loaded)
