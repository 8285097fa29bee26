"""An engine's loads run beside its compute step also where the streams that torch deals out in a row meet on one of the
runtime's four hardware queues."""
import ctypes

import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu
HELD = 20_000_000      # clocks that a stream is held for: 8 ms at 2.4 GHz, where a kernel or a small load takes 0.2 at most


def _beside(a, b):
    """Does a kernel on b end while one on a runs?"""
    import torch
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        torch.cuda._sleep(HELD)
        held = torch.cuda.Event()
        held.record()
    with torch.cuda.stream(b):
        x.add_(1)
    b.synchronize()
    beside = not held.query()
    torch.cuda.synchronize()
    return beside


def test_loads_run_beside_compute_whatever_streams_come(monkeypatch):
    import torch
    import paper_2410_03065_amd as cake
    streams = [torch.cuda.Stream() for _ in range(8)]
    for s in streams:
        _beside(torch.cuda.default_stream(), s)               # the first use binds a stream to its queue
    one_queue = next((a, b) for i, a in enumerate(streams) for b in streams[:i] if not _beside(a, b))
    coming = iter([*one_queue, *streams, *streams])
    shape = si.ModelShape("streams", 1, 256, 4, 2, 64, 256, 64, "bf16")
    with monkeypatch.context() as m:
        m.setattr(torch.cuda, "Stream", lambda device=None: next(coming))
        eng = cake.Engine(shape, None, max_tokens=128, max_chunk=64, page_tokens=64)
    eng.write_store(128, cake.STORE_INT8)                     # a copy and a kernel: the latter needs the hardware queue
    eng.load_chunk(0, 128)
    torch.cuda.synchronize()
    with torch.cuda.stream(eng.compute_stream):
        torch.cuda._sleep(HELD)
        step = torch.cuda.Event()
        step.record()
    eng.load_chunk(0, 128)
    ended_beside = not step.query()
    torch.cuda.synchronize()
    assert ended_beside


def test_streams_overlap():
    import torch
    import paper_2410_03065_amd as cake
    lib = cake.load_library()
    streams = [torch.cuda.Stream() for _ in range(6)]
    yes = ctypes.c_int32(7)

    def overlap(a, b):
        assert lib.cake_streams_overlap(a.cuda_stream, b.cuda_stream, ctypes.byref(yes)) == cake.OK
        return bool(yes.value)
    assert not overlap(streams[0], streams[0])
    found = [[a is not b and overlap(a, b) for b in streams] for a in streams]
    assert found == [[a is not b and _beside(a, b) for b in streams] for a in streams]
    assert sum(map(sum, found)) < 30                          # six streams on four queues: some meet
    assert lib.cake_streams_overlap(streams[0].cuda_stream, streams[1].cuda_stream, None) == cake.E_INVAL
