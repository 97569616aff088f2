"""The controller's stream ordering without a GPU: its calls run against a model
of two streams (the library's and torch's current one) that keeps, for every
operation, what is certain to have run before it."""
import contextlib
import importlib.util
import types

import numpy as np
import pytest
import torch

from paper_2409_07563_amd import _abi, controller


class Stream:
    """Operations in order; `seen[s]`: how many of stream s's precede the next one."""

    def __init__(self, handle):
        self.handle = self.cuda_stream = handle
        self.n, self.seen = 0, {}

    def run(self):
        self.n += 1
        return types.SimpleNamespace(stream=self, index=self.n, seen=dict(self.seen))

    def wait_stream(self, other):
        for s, n in {**other.seen, other: other.n}.items():
            self.seen[s] = max(self.seen.get(s, 0), n)

    def synchronize(self):
        pass


def before(a, b):
    if a.stream is b.stream:
        return a.index < b.index
    return b.seen.get(a.stream, 0) >= a.index


class Library:
    """The C ABI's calls as operations of the library's stream."""

    def __init__(self, world):
        self.world, self.ops = world, []

    def mppi_wait_stream(self, ctx, handle):
        self.world.lib.wait_stream(self.world.by_handle[handle])
        return 0

    def mppi_release_stream(self, ctx, handle):
        self.world.by_handle[handle].wait_stream(self.world.lib)
        return 0

    def mppi_put(self, ctx, what, ptr, handle):
        cur = self.world.by_handle[handle]
        cur.wait_stream(self.world.lib)
        self.ops.append(("mppi_put", cur.run()))
        self.world.lib.wait_stream(cur)
        return 0

    def mppi_theta_len(self, ctx):
        return 3

    def __getattr__(self, name):
        def call(*args):
            self.ops.append((name, self.world.lib.run()))
            return 0
        return call

    def last(self, name):
        return next(op for n, op in reversed(self.ops) if n == name)


@pytest.fixture
def world(monkeypatch):
    w = types.SimpleNamespace(lib=Stream(11), cur=Stream(22), capturing=False)
    w.by_handle = {22: w.cur}
    monkeypatch.setattr(controller, "_raw_stream", lambda device: w.cur.handle)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: w.cur)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: w.capturing)
    monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())
    c = object.__new__(controller.Controller)
    c.device = torch.device("cpu")
    c.stream, c.ctx, c._lib = w.lib, 1, Library(w)
    c.batch, c.requires_grad, c.n_inst, c.T, c.m, c.K = False, True, 1, 4, 2, 8
    c._captured = {}
    c._joined, c._home = False, torch.device("cpu", 0)
    c._off = {k: np.array([0, n]) for k, n in ((_abi.PACKED_STATE, 4), (_abi.PACKED_CONTROLS, 8),
                                               (_abi.PACKED_SAMPLES, 8), (_abi.PACKED_NOISE, 64))}
    w.ctl = c
    yield w
    c.ctx = None


OWN = {"mppi_shift": lambda c: c.shift(1), "mppi_sample": lambda c: c.sample(),
       "mppi_rollout": lambda c: c.rollout(), "mppi_update": lambda c: c.update(),
       "mppi_iterate": lambda c: c.iterate(2), "mppi_set_iteration": lambda c: c.set_iteration(3),
       "mppi_set_theta": lambda c: c.set_theta(np.ones(3))}


@pytest.mark.parametrize("name", sorted(OWN))
def test_eager_calls_and_replays_follow_each_other(world, name):
    """Once a call was captured, a replay (work of the caller's stream on the
    context's buffers) is ordered with every eager call around it."""
    c = world.ctl
    world.capturing = True
    c.iterate(1)
    world.capturing = False
    replay = world.cur.run()
    OWN[name](c)
    call = c._lib.last(name)
    assert before(replay, call)
    assert before(call, world.cur.run())


def test_calls_of_a_context_never_captured_order_nothing(world):
    c = world.ctl
    first = world.cur.run()
    c.iterate(1)
    assert not before(first, c._lib.last("mppi_iterate"))
    assert not before(c._lib.last("mppi_iterate"), world.cur.run())


def test_close_waits_for_replays(world):
    c = world.ctl
    world.capturing = True
    c.sample()
    world.capturing = False
    replay = world.cur.run()
    c.close()
    assert before(replay, c._lib.last("mppi_destroy"))


def test_a_controller_of_another_device(world, monkeypatch):
    """The controller's device is 1 while device 0 is current: the stream it is
    ordered with and the capture it joins are device 1's."""
    c = world.ctl
    c.device, c._home = torch.device("cuda"), torch.device("cuda", 1)
    other, asked = Stream(33), []
    world.by_handle[33] = other
    now = [0]

    @contextlib.contextmanager
    def device(d):
        old, now[0] = now[0], d.index
        yield
        now[0] = old

    monkeypatch.setattr(torch.cuda, "current_device", lambda: now[0])
    monkeypatch.setattr(torch.cuda, "device", device)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing",
                        lambda: asked.append(now[0]) or (world.capturing and now[0] == 1))
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda d=None: other if (now[0] if d is None else d.index) == 1 else world.cur)
    monkeypatch.setattr(controller, "_raw_stream", lambda d: {0: 22, 1: 33}[d])
    monkeypatch.setattr(torch, "empty", lambda shape, dtype=None, device=None:
                        types.SimpleNamespace(device=device, data_ptr=lambda: 0, reshape=lambda *a: 0,
                                              view=lambda *a: 0))
    first = other.run()
    c.controls()
    read = c._lib.last("mppi_get_controls")
    assert before(first, read) and before(read, other.run())
    assert not before(read, world.cur.run())
    world.capturing = True
    second = other.run()
    c.iterate(1)
    assert before(second, c._lib.last("mppi_iterate"))
    assert set(asked) == {1}


INPUTS = {"mppi_set_state": (4, lambda c, t: c.set_state(t)),
          "mppi_set_controls": (8, lambda c, t: c.set_controls(t)),
          "mppi_set_costs": (8, lambda c, t: c.set_costs(t))}
FORMS = {"as it is": lambda n: torch.zeros(n), "binary64": lambda n: torch.zeros(n).double(),
         "strided": lambda n: torch.zeros(2 * n)[::2]}


@pytest.mark.parametrize("captured", [False, True])
@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("name", sorted(INPUTS))
def test_an_input_may_be_written_after_the_call(world, name, form, captured):
    """What the caller's stream does next, such as reusing the tensor's memory,
    follows the read (and the conversion before it)."""
    n, call = INPUTS[name]
    c, t = world.ctl, FORMS[form](n)
    made = world.cur.run()
    world.capturing = captured
    c.iterate(5)
    call(c, t)
    read = c._lib.last(name if captured else "mppi_put")
    long = c._lib.last("mppi_iterate")
    assert before(made, read) and before(long, read)
    assert before(read, world.cur.run())
    c.iterate(1)
    assert before(read, c._lib.last("mppi_iterate"))


def test_a_torch_without_the_raw_stream_function(monkeypatch):
    """The package loads, and takes the handle from the current stream."""
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda device: types.SimpleNamespace(cuda_stream=100 + device))
    spec = importlib.util.spec_from_file_location("paper_2409_07563_amd._controller_again",
                                                  controller.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    assert again._raw_stream(1) == 101
