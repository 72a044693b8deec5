"""The forward call in native code (csrc/dfa_torch.cpp) against the one that Python marshals: the same results bit for bit from the
same kernels, whichever of them a call's arguments lead to, and the same refusals."""
import numpy as np
import pytest

from gpu_util import make_qkv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2403_09195_amd import binding
    binding.lib()
    return binding


def _python(B, monkeypatch, *args, **kw):
    with monkeypatch.context() as m:
        m.setattr(B, "_native_forward", lambda *a: None)
        return B.forward(*args, **kw)


# short, split (its workspace comes from the callback) and whole-tile launches, fp32; packed strides; a table of offsets
@pytest.mark.parametrize("N,branches,table", [(200, [(50, 1), (200, 4)], False), (4096, [(1024, 1), (2048, 2), (4096, 4)], False),
                                              (4096, [(4096, 1)], False), (300, [(100, 1), (150, 3)], True)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_same_results(B, monkeypatch, N, branches, table, dtype):
    import torch
    (q, k, v), _ = make_qkv(21, 1, N, 4, 64, dtype)
    q, k, v = torch.stack((q, k, v), dim=2).unbind(2)
    offsets = [[(h + x) % r for h in range(4)] for x, (_, r) in enumerate(branches)] if table else None
    native = B._native_forward(q, k, v, branches, 0.125, offsets)
    assert type(native) is tuple
    for other in (_python(B, monkeypatch, q, k, v, branches, 0.125, head_offsets=offsets),
                  B.forward(q, k, v, tuple(branches), 0.125, head_offsets=offsets)):
        assert all(torch.equal(a, b) and a.dtype == b.dtype and a.shape == b.shape and a.is_contiguous() for a, b in zip(native, other))


# The backward: short and whole-tile launches, fp32; packed strides; a table of offsets; gradients and results that Python refuses stay refused.
@pytest.mark.parametrize("Bsz,N,branches,table", [(1, 200, [(50, 1), (200, 4)], False), (64, 128, [(128, 1)], False), (2, 300, [(100, 1), (150, 3)], True)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_backward_same_results(B, monkeypatch, Bsz, N, branches, table, dtype):
    import torch
    (q, k, v), _ = make_qkv(25, Bsz, N, 4, 64, dtype)
    dout = v.flip(1).contiguous()
    q, k, v = torch.stack((q, k, v), dim=2).unbind(2)
    offsets = [[(h + x) % r for h in range(4)] for x, (_, r) in enumerate(branches)] if table else None
    out, lse = B.forward(q, k, v, branches, 0.125, head_offsets=offsets)
    native = B._native_backward(q, k, v, out, lse, dout, branches, 0.125, offsets)
    assert type(native) is tuple and B._native_backward(q, k, v, out, lse, dout, branches, 1, offsets) is None
    with monkeypatch.context() as m:
        m.setattr(B, "_native_backward", lambda *a: None)
        python = B.backward(q, k, v, out, lse, dout, branches, 0.125, head_offsets=offsets)
    for other in (python, B.backward(q, k, v, out, lse, dout, tuple(branches), 0.125, head_offsets=offsets)):
        assert all(torch.equal(a, b) and a.dtype == b.dtype and a.shape == b.shape and a.is_contiguous() for a, b in zip(native, other))
    for bad, error in ((dict(dout=dout.transpose(1, 2)), ValueError), (dict(lse=lse.double()), TypeError), (dict(out=out.half()), TypeError),
                       (dict(dout=dout.cpu()), RuntimeError), (dict(k=k[:, :-1]), B.DfaError), (dict(branches=[(64, 0)]), B.DfaError)):
        with pytest.raises(error):
            B.backward(**{**dict(q=q, k=k, v=v, out=out, lse=lse, dout=dout, branches=branches, scale=0.125, head_offsets=offsets), **bad})


# out, lse and dout that hold less than the call reads, or something else in its order, are refused on both paths before anything is launched; what
# holds more, or the same without all dimensions, is read as ever.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Bsz", [1, 2])
def test_backward_refuses_what_it_would_read_past(B, monkeypatch, Bsz, dtype):
    import torch
    N, H, D, branches = 96, 4, 64, [(48, 1), (96, 3)]
    (q, k, v), _ = make_qkv(26, Bsz, N, H, D, dtype)
    out, lse = B.forward(q, k, v, branches, 0.125)
    dout = v.flip(1).contiguous()
    call = lambda **kw: B.backward(**{**dict(q=q, k=k, v=v, out=out, lse=lse, dout=dout, branches=branches, scale=0.125), **kw})
    ref = call()
    flat = lambda t, *shape: t.reshape(shape)
    twice = lambda t: torch.cat((t, t))
    bad = [(name, b) for name, t in (("out", out), ("dout", dout)) for b in
           (t[:, :-1].contiguous(), t[:, :, :-1].contiguous(), t[:, :, :, :32].contiguous(), t[:0], t.transpose(1, 2).contiguous(), flat(t, -1)[:-64],
            t[:, :N // 2].contiguous(), torch.empty((Bsz, N, 2 * H, D), dtype=t.dtype, device="cuda"))]
    bad += [("lse", b) for b in (lse[:, :, :-1].contiguous(), lse[:, :-1].contiguous(), lse.transpose(1, 2).contiguous(), lse[:0], flat(lse, -1)[:-1],
                                 torch.empty((Bsz, H, 2 * N), device="cuda"))]
    if Bsz > 1:
        bad += [("out", out[:1]), ("dout", dout[:1]), ("lse", lse[:1]), ("dout", torch.cat((dout, dout), dim=1))]
    good = [("out", twice(out)), ("dout", twice(dout)), ("lse", twice(lse)), ("dout", flat(dout, Bsz, N, H * D)), ("out", flat(out, -1)),
            ("lse", flat(lse, Bsz * H, N))]
    if Bsz == 1:
        good += [("dout", torch.cat((dout, dout), dim=1)), ("lse", torch.cat((lse, lse), dim=1))]
    native = B._native_backward
    for path in (native, lambda *a: None):
        monkeypatch.setattr(B, "_native_backward", path)
        for name, t in bad:
            assert t.is_contiguous()
            with pytest.raises(B.DfaError):
                call(**{name: t})
        for name, t in good:
            assert all(torch.equal(a, b) for a, b in zip(ref, call(**{name: t}))), (name, tuple(t.shape))
    for name, t in good:                       # and the native call takes them itself
        args = {**dict(out=out, lse=lse, dout=dout), name: t}
        assert type(native(q, k, v, args["out"], args["lse"], args["dout"], branches, 0.125, None)) is tuple


def test_calls_left_to_python(B):
    import torch
    (q, k, v), _ = make_qkv(22, 1, 64, 2, 64, "bf16")
    ref = B.forward(q, k, v, [(64, 1)], 0.125)
    for branches, scale, offsets in (([(np.int64(64), 1)], 0.125, None), ([(64, 1)], np.float32(0.125), None),
                                     ([(64, 1)], 0.125, np.zeros((1, 2), dtype=np.int32))):
        assert B._native_forward(q, k, v, branches, scale, offsets) is None
        assert all(torch.equal(a, b) for a, b in zip(ref, B.forward(q, k, v, branches, scale, head_offsets=offsets)))
    out, lse = B.forward(q, k, v, [(64, 1)], 0.125, want_lse=False)
    assert lse is None and torch.equal(out, ref[0])


def test_refusals(B):
    import torch
    (q, k, v), _ = make_qkv(23, 1, 64, 2, 64, "bf16")
    for bad, code in (([(64, 0)], -2), ([(0, 1)], -2)):
        with pytest.raises(B.DfaError) as e:
            B.forward(q, k, v, bad, 0.125)
        assert e.value.code == code
    with pytest.raises(B.DfaError):
        B.forward(q, k, v, [(64, 1)] * 9, 0.125)
    with pytest.raises(B.DfaError):
        B.forward(q, k, v, [(64, 1)], 0.0)
    with pytest.raises(B.DfaError):
        B.forward(q.half(), k.half(), v.half(), [(64, 1)], 0.125)
    with pytest.raises(RuntimeError):
        B.forward(q.cpu(), k, v, [(64, 1)], 0.125)
    with pytest.raises(B.DfaError):
        B.forward(q.transpose(2, 3), k, v, [(64, 1)], 0.125)


def test_side_stream(B):
    """The launch goes to the current stream: there q is filled only after a wait of some milliseconds, and any other stream is idle."""
    import torch
    (q, k, v), _ = make_qkv(24, 1, 1024, 4, 64, "bf16")
    ref = B.forward(q, k, v, [(256, 1)], 0.125)
    q2 = torch.zeros_like(q)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        q2.copy_(q)
        out, lse = B.forward(q2, k, v, [(256, 1)], 0.125)
        assert not side.query(), "the stream had nothing left to wait for"
    side.synchronize()
    assert torch.equal(out, ref[0]) and torch.equal(lse, ref[1])


def test_other_threads_run_during_a_call(B):
    """The first call of a shape builds its plan, about a second here: other threads are not held up by it."""
    import threading
    import time
    import torch
    q, k, v = torch.randn((3, 1, 65536, 4, 64), device="cuda").bfloat16().unbind(0)
    branches = [(50, 1), (1000, 3), (65536, 5)]
    torch.cuda.synchronize()
    ticks, stop = [], threading.Event()

    def tick():
        while not stop.is_set():
            ticks.append(time.monotonic())
            time.sleep(0.001)

    thread = threading.Thread(target=tick)
    thread.start()
    try:
        while not ticks:
            time.sleep(0.001)
        B.release_plans()
        t0 = time.monotonic()
        assert type(B._native_forward(q, k, v, branches, 0.125, None)) is tuple
        t1 = time.monotonic()
    finally:
        stop.set()
        thread.join()
    during = [t for t in ticks if t0 <= t <= t1]
    assert t1 - t0 > 0.05, "the call was too short to tell"
    assert len(during) > 10, (len(during), t1 - t0)


def test_keys_and_values_smaller_than_q(B):
    """The native call hands them back, and every entry point refuses them."""
    import torch
    (q, k, v), _ = make_qkv(25, 2, 64, 2, 64, "bf16")
    (qf, _, _), _ = make_qkv(25, 2, 64, 2, 64, "f32")
    for bad, code in ((k[:1], -2), (k[:, :32], -2), (k[:, :, :1], -2), (qf, -4)):
        for kk, vv in ((bad, v), (k, bad)):
            assert B._native_forward(q, kk, vv, [(64, 1)], 0.125, None) is None
            for call in (lambda: B.forward(q, kk, vv, [(64, 1)], 0.125), lambda: B.forward_static(q, kk, vv, [(64, 1)], 0.125),
                         lambda: B.forward_branch(q, kk, vv, 64, 1, 0.125), lambda: B.backward(q, kk, vv, q, torch.zeros((2, 2, 64), device="cuda"), q, [(64, 1)], 0.125)):
                with pytest.raises(B.DfaError) as e:
                    call()
                assert e.value.code == code
    ref = B.forward(q, k, v, [(64, 1)], 0.125)
    longer = torch.cat((k, k), dim=1)
    assert all(torch.equal(a, b) for a, b in zip(ref, B.forward(q, longer, v, [(64, 1)], 0.125)))
