"""Order of the wrapper's calls with the caller's stream, from a record of
the stream operations (no GPU): a batch works on a stream of its own, so it
has to wait for the caller's before it reads or writes a tensor of the
caller's, the allocator has to know of every such use that may still run
when the tensor is dropped, and a caller's stream that goes on to read a
result has to wait for the batch."""

import pytest
import torch

from paper_1909_01580_amd import hgks


class Stream:
    def __init__(self, name, log):
        self.name, self.log, self.cuda_stream, self.stream_id = name, log, 0, id(self)

    def wait_stream(self, other):
        self.log.append(("wait", self.name, other.name))

    def synchronize(self):
        self.log.append(("host waits", self.name))


class Tensor:
    """Stands for a device tensor of the caller's."""

    def __init__(self, name, log):
        self.name, self.log = name, log

    def record_stream(self, stream):
        self.log.append(("record", self.name, stream.name))

    def numel(self):
        return 0

    def data_ptr(self):
        return 0

    def __getitem__(self, _):
        return self


@pytest.fixture
def world(monkeypatch):
    """(log, own stream, caller's stream): every library call and stream operation in order."""
    log = []
    own, caller = Stream("own", log), Stream("caller", log)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: caller)
    monkeypatch.setattr(torch.accelerator, "current_stream", lambda device=None: caller)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(torch, "empty", lambda *a, **k: Tensor("new", log))
    for name in hgks.EXPORTS:
        if hasattr(hgks, name) and name != "hgks_default_config":
            monkeypatch.setattr(hgks, name, lambda *a, _n=name, **k: log.append(("call", _n)) or 0)
    return log, own, caller


def batch(own):
    b = object.__new__(hgks.Batch)
    b.device, b.stream, b.h, b.n, b.grids = torch.device("cpu"), own, None, 1, [{"n": (4, 4, 4)}]
    return b


CALLER_FIRST = ("wait", "own", "caller")


def test_batch_get_state_waits_for_the_caller(world):
    """The output's memory may have been dropped by the caller with work on
    it still queued; the host, which waits for the copy, may do the waiting."""
    log, own, _ = world
    batch(own).get_state(0)
    copy = log.index(("call", "hgks_batch_get_state"))
    assert CALLER_FIRST in log[:copy] or ("host waits", "caller") in log[:copy]
    assert ("call", "hgks_batch_sync") in log[copy:]


def test_batch_step_waits_for_the_time_steps_and_keeps_them(world):
    log, own, _ = world
    batch(own).step(Tensor("dt", log))
    launch = log.index(("call", "hgks_batch_step"))
    assert CALLER_FIRST in log[:launch]
    assert ("record", "dt", "own") in log[launch:]


def test_batch_max_dt_orders_both_streams(world):
    log, own, _ = world
    batch(own).max_dt(0.35, Tensor("dt", log))
    launch = log.index(("call", "hgks_batch_max_dt"))
    assert CALLER_FIRST in log[:launch]
    assert ("record", "dt", "own") in log[launch:] and ("wait", "caller", "own") in log[launch:]
    # into the batch's own array: nothing of the caller's is touched
    del log[:]
    batch(own).max_dt(0.35)
    assert log == [("call", "hgks_batch_max_dt")]


def test_batch_workspace_belongs_to_its_stream(world):
    """The workspace comes from the caller's stream's allocator, is written
    by the batch's stream, and may be dropped while that still runs."""
    log, own, _ = world
    hgks.Batch([{"n": (4, 4, 4), "length": (1.0, 1.0, 1.0)}], device="cpu", stream=own)
    create = log.index(("call", "hgks_batch_create"))
    assert CALLER_FIRST in log[:create]
    assert ("record", "new", "own") in log


def test_one_stream_needs_no_order(world):
    log, _, caller = world
    b = batch(caller)
    b.step(Tensor("dt", log))
    b.max_dt(0.35, Tensor("dt", log))
    b.get_state(0)
    assert not [e for e in log if e[0] in ("wait", "host waits")]


def test_nothing_is_ordered_while_the_caller_is_captured(world, monkeypatch):
    """A wait would draw the batch's own stream into the caller's capture,
    and its calls, which run at once as ever, would be refused there."""
    log, own, _ = world
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    b = batch(own)
    b.step(Tensor("dt", log))
    b.max_dt(0.35, Tensor("dt", log))
    b.get_state(0)
    assert not [e for e in log if e[0] in ("wait", "host waits")]


def context(own):
    c = object.__new__(hgks.Context)
    c.device, c.stream, c.h, c.n = torch.device("cpu"), own, None, (4, 4, 4)
    return c


@pytest.mark.parametrize("method,args,written", [
    ("set_state", 1, False), ("set_vertices", 2, False), ("set_next_vertices", 1, False),
    ("get_state", 1, True), ("get_state", 0, True), ("debug_fallback_mask", 0, True),
    ("debug_gp_states", 0, True), ("debug_face_flux", 0, True)])
def test_context_on_another_stream(world, method, args, written):
    """A context given a stream of its own, called under the caller's."""
    log, own, caller = world
    t = Tensor("t", log)
    call = (t, (1.0,) * 3)[:args] if method.startswith(("set", "get")) else (1e-3,)
    getattr(context(own), method)(*call)
    launch = log.index(("call", "hgks_" + method))
    assert CALLER_FIRST in log[:launch]
    assert ("record", "t" if args else "new", "own") in log[launch:]
    assert (("wait", "caller", "own") in log[launch:]) == written
    # the usual case, one stream: the library call alone
    del log[:]
    getattr(context(caller), method)(*call)
    assert log == [("call", "hgks_" + method)]


def test_context_workspace_belongs_to_its_stream(world):
    log, own, _ = world
    hgks.Context((4, 4, 4), device="cpu", stream=own)
    assert CALLER_FIRST in log[:log.index(("call", "hgks_create"))]
    assert ("record", "new", "own") in log
