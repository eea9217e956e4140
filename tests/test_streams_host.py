"""CPU test of the stream that the front end's own buffers belong to: with stand-ins for torch's streams and for the
library's device entry points, every buffer that a call with `stream` allocates is allocated on that stream, and what
the call returns is recorded on the current one."""
import contextlib

import numpy as np
import pytest

from paper_2402_04834_amd import _lib, workload

DEVICE_CALLS = ("bbp_decode_device", "bbp_decode_device_noalloc", "bbp_decode_groups", "bbp_autotune",
                "bbp_bmps_decode_device", "bbp_warm_predict", "bbp_warm_loss_grad", "bbp_warm_decode")


class Stream:
    def __init__(self, name):
        self.name, self.cuda_stream, self.waited = name, 1, []

    def wait_stream(self, other):
        self.waited.append(other.name)


class Library:
    """The library's host functions; its device entry points only note the stream they were called for."""

    def __init__(self, real):
        self.real = real

    def __getattr__(self, name):
        return (lambda *a: 0) if name in DEVICE_CALLS else getattr(self.real, name)


@pytest.fixture
def world(monkeypatch):
    import torch

    class Cuda(torch.Tensor):   # a CPU tensor that claims to be the GPU's
        is_cuda = property(lambda self: True)

    log = dict(active=Stream("current"), made={}, recorded={}, summed=[])

    @contextlib.contextmanager
    def use_stream(s):
        before = log["active"]
        log["active"] = s if s is not None else before
        yield
        log["active"] = before

    def noting(make):
        def f(*a, **kw):
            t = make(*a, **kw)
            log["made"][t.data_ptr()] = (log["active"].name, t)   # kept: no address comes twice
            return t
        return f

    total = torch.Tensor.sum
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev=None: log["active"])
    monkeypatch.setattr(torch.cuda, "stream", use_stream)
    for name in ("empty", "zeros", "empty_like", "zeros_like"):
        monkeypatch.setattr(torch, name, noting(getattr(torch, name)))
    monkeypatch.setattr(torch.Tensor, "record_stream",
                        lambda t, s: log["recorded"].setdefault(t.data_ptr(), []).append(s.name))
    monkeypatch.setattr(torch.Tensor, "sum", lambda t, *a: (log["summed"].append(log["active"].name), total(t, *a))[1])
    lib = Library(_lib.lib())
    monkeypatch.setattr(_lib, "lib", lambda: lib)
    log["cuda"] = lambda x: torch.from_numpy(np.ascontiguousarray(x)).as_subclass(Cuda)
    return log


def _calls():
    import torch
    import paper_2402_04834_amd as bbp
    from paper_2402_04834_amd import warm
    d, b = 5, 2
    opts = bbp.default_opts(block=3, chi=32)
    M = bbp.plan_query(d, opts).num_messages
    _, syn = workload.make_batch(d, 0.1, b)
    theta = warm.init_params(1)
    targets = np.ones((b, 4, M, 64), dtype=np.float32)

    def loss(w, st, use):
        return warm.loss_grad(d, 0.1, w["cuda"](syn), opts, torch.from_numpy(theta), torch.from_numpy(targets),
                              torch.from_numpy(np.full(4 * b, use, dtype=np.uint8)), stream=st)

    return {
        "decode_device": lambda w, st: bbp.decode_device(d, 0.1, w["cuda"](syn), opts, messages=True, stream=st),
        "decode_device_noalloc": lambda w, st: bbp.decode_device_noalloc(d, 0.1, w["cuda"](syn), opts, stream=st),
        "decode_groups": lambda w, st: bbp.decode_groups([(d, 0.1, w["cuda"](syn))], opts, messages=True, stream=st),
        "bmps_decode": lambda w, st: bbp.bmps_decode(d, 0.1, w["cuda"](syn), 4, stream=st),
        "autotune": lambda w, st: bbp.autotune(d, 0.1, w["cuda"](syn), opts, stream=st),
        "predict": lambda w, st: warm.predict(d, 0.1, w["cuda"](syn), opts, torch.from_numpy(theta), stream=st),
        "loss_grad": lambda w, st: loss(w, st, 1),
        "loss_grad unused": lambda w, st: loss(w, st, 0),
        "warm decode": lambda w, st: warm.decode(d, 0.1, w["cuda"](syn), opts, torch.from_numpy(theta), stream=st),
    }


def _tensors(x):
    import torch
    if isinstance(x, torch.Tensor):
        yield x
    elif isinstance(x, (list, tuple, dict)):
        for y in (x.values() if isinstance(x, dict) else x):
            yield from _tensors(y)


@pytest.mark.parametrize("name", ["decode_device", "decode_device_noalloc", "decode_groups", "bmps_decode", "autotune",
                                  "predict", "loss_grad", "loss_grad unused", "warm decode"])
def test_buffers_belong_to_the_stream_of_the_call(world, name):
    call = _calls()[name]
    world["made"].clear()
    side = Stream("side")
    result = call(world, side)
    assert world["made"] and {s for s, _ in world["made"].values()} == {"side"}
    for t in _tensors(result):
        assert world["recorded"].get(t.data_ptr()) == ["current"]
    if name.startswith("loss_grad"):   # `use` is read in the stream's order, after what the current one holds
        assert world["summed"] == ["side"] and side.waited == ["current"]
