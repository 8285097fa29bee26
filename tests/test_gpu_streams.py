"""An engine's loads run beside its compute step also where the streams that torch deals out in a row meet on one of the
runtime's four hardware queues, and so do the compute steps of three engines in turn; and its ops wait for operands that
torch's stream has yet to write."""
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


def test_engines_in_turn_compute_side_by_side():
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("streams", 1, 256, 4, 2, 64, 256, 64, "bf16")
    engines = [cake.Engine(shape, None, max_tokens=128, max_chunk=64, page_tokens=64) for _ in range(6)]
    for k, e in enumerate(engines):
        assert _beside(e.compute_stream, e.copy_stream)
        for other in engines[max(0, k - 2):k]:
            assert _beside(e.compute_stream, other.compute_stream)


def test_ops_wait_for_their_operands():
    import torch
    import paper_2410_03065_amd as cake
    shape = si.ModelShape("operands", 1, 256, 4, 2, 64, 256, 64, "bf16")
    while True:                                               # on one hardware queue they would wait by chance
        eng = cake.Engine(shape, None, max_tokens=128, max_chunk=64, page_tokens=64, with_head=True)
        if _beside(torch.cuda.default_stream(), eng.compute_stream):
            break
    eng.pool.normal_()
    rnd = lambda dtype, *dims: torch.randn(*dims, device="cuda").to(dtype)
    bf, f32 = torch.bfloat16, torch.float32
    a, w, x, q, q1, qkv = rnd(bf, 64, 256), rnd(bf, 256, 256), rnd(f32, 64, 256), rnd(bf, 4, 64, 64), rnd(f32, 4, 64), rnd(f32, 64, 512)
    gain = torch.ones(256, device="cuda")
    ops = {"rmsnorm": (x, lambda t: eng.op_rmsnorm(t, gain)), "gemm": (a, lambda t: eng.op_gemm(t, w)),
           "gemm_residual": (a, lambda t: eng.op_gemm_residual(t, w, x.clone())), "gemm_swiglu": (a, lambda t: eng.op_gemm_swiglu(t, w, w)),
           "attention": (q, lambda t: eng.op_attention(t, 0, 0)), "decode_attention": (q1, lambda t: eng.op_decode_attention(t, 0, 128)),
           "rope_kv_write": (qkv, lambda t: eng.op_rope_kv_write(t, 0, 64))}   # last: it writes to the pool
    wrong = []
    for name, (operand, op) in ops.items():
        torch.cuda.synchronize()
        want = op(operand).clone()
        late = torch.zeros_like(operand)
        torch.cuda.synchronize()
        torch.cuda._sleep(HELD)
        late.copy_(operand)
        got = op(late)
        torch.cuda.synchronize()
        assert float(want.abs().max()) > 0
        if not torch.equal(got, want):
            wrong.append(name)
    assert not wrong, wrong
