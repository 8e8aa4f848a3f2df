"""The step's workspaces (``step.Replica``), checked on the CPU: no call of a step, however its work is
placed, needs more than the workspace it is handed.  A call given too little makes a temporary of its
own; from a recorded program that memory would be written again after it was freed.

The replica is built on the CPU over the library's own workspace queries; every other library call is
replaced by one that does nothing.
"""
import gc
import weakref

import pytest
import torch

from paper_1605_08695_amd import ops, step, workloads as W
from paper_1605_08695_amd._lib import load


def two_branches(k, n=32, hw=28, cin=256, concat=False):
    """Two 1x1 branches that read one tensor (run as one merged convolution), each followed by a k x k
    convolution into a concat.  The tensor is the input, or, with ``concat``, a concat, whose last
    reader's input gradient applies the concat's ReLU backward."""
    b = W._Builder("two_branches_%dx%d" % (k, k), "bf16", 1e-6, not concat, (n, hw, hw, cin))
    src = "x"
    if concat:
        src = b.concat_buffer("x", (hw, hw), cin)
        b.conv("x", cin // 2, 1, dst=src, c0=0, name="s0")
        b.conv("x", cin // 2, 1, dst=src, c0=cin // 2, name="s1")
    cat = b.concat_buffer(src, (hw, hw), 64)
    p = (k // 2,) * 4
    for i in range(2):
        r = b.conv(src, 64, 1, name="r%d" % i)
        b.conv(r, 32, k, pads=p, dst=cat, c0=32 * i, name="b%d" % i)
    return b.done(cat)


NETS = [("two_1x1", lambda: two_branches(1)), ("two_3x3", lambda: two_branches(3)),
        ("two_of_concat", lambda: two_branches(3, n=2, hw=14, concat=True)),
        ("single_layer", lambda: W.single_layer(batch=2, hw=16)), ("alexnet", lambda: W.alexnet(batch=2)),
        ("googlenet", lambda: W.googlenet(batch=2)), ("inception_v3", lambda: W.inception_v3(batch=1)),
        ("classifier", lambda: W.classifier_small(batch=2, dtype="bf16"))]


class _Stream:
    cuda_stream = 0


class _Lib:
    """The library's workspace queries; every other call succeeds and does nothing."""

    def __getattr__(self, name):
        return getattr(load(), name) if name.endswith("_workspace_bytes") else lambda *a: 0


@pytest.fixture
def cpu_replica(monkeypatch):
    monkeypatch.setattr(ops, "load", _Lib)
    monkeypatch.setattr(ops, "_stream", lambda stream: 0)
    monkeypatch.setattr(step, "_device_streams", lambda dev, n: [_Stream() for _ in range(n)])
    monkeypatch.setattr(step, "_capture_stream", lambda dev, shared: _Stream())
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: _Stream())
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)

    def temporary(nbytes, device, stream=None):
        raise AssertionError("a call of the step needs a temporary workspace of %d bytes" % nbytes)
    monkeypatch.setattr(ops, "_ws", temporary)
    return lambda net, **kw: step.Replica(net, W.make_inputs(net, seed=0), device="cpu", **kw)


@pytest.mark.parametrize("name,make", NETS, ids=[n for n, _ in NETS])
def test_no_call_of_a_step_needs_a_temporary(cpu_replica, name, make):
    net = make()
    for merge in (True, False):
        rep = cpu_replica(net, merge=merge)
        for streams in (False, True):
            for defer in (True, False):
                rep.use_streams, rep.defer_bias = streams, defer
                rep.step()
        rep.step(trace=lambda event, op, stream=None, **kw: None)
        rep.step(concurrent=False)


def test_recorded_program_keeps_what_its_calls_allocate(monkeypatch):
    """Workspaces and results that recorded calls made themselves live as long as their program, whose
    runs write them again; unrecorded ones are freed on return."""
    made, empty = [], torch.empty

    def tracked(*args, **kw):
        t = empty(*args, **kw)
        made.append(weakref.ref(t))
        return t
    monkeypatch.setattr(ops, "load", _Lib)
    monkeypatch.setattr(ops, "_stream", lambda stream: 0)
    x, dy, w = torch.zeros(32, 28, 28, 64), torch.zeros(32, 28, 28, 64), torch.zeros(1, 1, 64, 64)
    monkeypatch.setattr(torch, "empty", tracked)

    def calls():
        ops.conv2d_bwd_filter(x, dy, (1, 1), 1, (0, 0, 0, 0))
        ops.conv2d_bwd_input_relu_bwd(dy, w, x, torch.zeros_like(x), 1, (0, 0, 0, 0))
        gc.collect()
        return [r() is not None for r in made]
    assert len(calls()) == 4 and not any(calls())
    made.clear()
    prog = ops.Program()
    with prog.recording():
        alive = calls()
    assert len(alive) == 4 and all(alive)
    with pytest.raises(ZeroDivisionError), ops.Program().recording():
        1 / 0
    assert all(r() is not None for r in made)
    first = list(made)
    with prog.recording():                  # recorded anew: the earlier calls are gone, and their memory
        calls()
    assert not any(r() is not None for r in first)
    prog.close()
    gc.collect()
    assert not any(r() is not None for r in made)
    made.clear()
    assert not any(calls())
