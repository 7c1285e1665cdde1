"""Tensors that a batch's own stream and the caller's stream share, with work
still queued on one of them when the other takes over.  Every comparison is
of the same bits, with the result of the same calls one after another."""

import pytest
import torch

from tests.helpers import smooth_state

pytestmark = pytest.mark.gpu

N, L = (32, 24, 20), (3.2, 2.4, 2.0)
DEV = "cuda:0"


@pytest.fixture(scope="module")
def hg():
    from paper_1909_01580_amd import hgks
    hgks.load()
    return hgks


@pytest.fixture(scope="module")
def busy():
    """Queues some tens of milliseconds of work on the current stream."""
    a = torch.ones(4096, 4096, dtype=torch.float64, device=DEV)

    def queue():
        b = a
        for _ in range(20):
            b = a @ a
        return b
    queue()
    torch.cuda.synchronize()
    return queue


def state(seed):
    return torch.tensor(smooth_state(N, L, seed, mach=0.5), device=DEV)


def batch(hg, q, **kw):
    b = hg.Batch([{"n": N, "length": L, "mu": 0.0}], precision="fp64", **kw)
    b.set_state(0, q)
    return b


def test_get_state_does_not_take_memory_in_use(hg, busy):
    """Snapshots as a program takes them: each state is converted on the
    caller's stream and dropped, with the conversion still waiting when the
    next state is asked for, which gets the dropped one's memory."""
    qs = [state(s) for s in range(6)]
    b = hg.Batch([{"n": N, "length": L, "mu": 0.0}] * 6, precision="fp64")
    for i, q in enumerate(qs):
        b.set_state(i, q)
    b.sync()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    for _ in range(3):
        busy()
        got, where = [], []
        for i in range(6):
            q = b.get_state(i)
            where.append(q.data_ptr())
            busy()
            got.append(q.float())
            del q
        assert len(set(where)) < 6, "the allocator reused no memory: nothing was tested"
        for q, g in zip(qs, got):
            assert torch.equal(g, q.float())


def test_step_reads_time_steps_still_being_written_and_then_dropped(hg, busy):
    q = state(7)
    dt = 1e-3
    ref = batch(hg, q)
    kept = torch.tensor([dt], dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    for _ in range(4):
        ref.step(kept, 2)
    want = ref.get_state(0)
    b = batch(hg, q)
    for _ in range(4):
        busy()
        t = torch.zeros(1, dtype=torch.float64, device=DEV)
        t += dt                                   # behind the queue on the caller's stream
        with torch.cuda.stream(b.stream):
            busy()                                # the step starts long after its call
        b.step(t, 2)
        del t
        junk = [torch.full((1,), 1e3, dtype=torch.float64, device=DEV) for _ in range(64)]
    assert torch.equal(b.get_state(0), want)
    del junk


def test_max_dt_is_read_on_the_callers_stream(hg, busy):
    q = state(8)
    b = batch(hg, q)
    b.max_dt(0.35)
    want = b.dt()
    for _ in range(3):
        t = torch.zeros(1, dtype=torch.float64, device=DEV)
        with torch.cuda.stream(b.stream):
            busy()
        b.max_dt(0.35, t)
        assert (t * 1.0).tolist() == want


def test_workspace_of_a_dropped_batch(hg, busy):
    """A batch dropped with its steps still queued keeps its workspace until they ran."""
    q = state(9)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    b = batch(hg, q)
    b.sync()
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device=DEV)
    size = b.workspace.numel()
    with torch.cuda.stream(b.stream):
        busy()
    for _ in range(3):
        b.step(dt, 2)
    del b
    fresh = [torch.zeros(size, dtype=torch.uint8, device=DEV) for _ in range(2)]
    torch.cuda.synchronize()
    assert not any(f.any() for f in fresh)


def test_step_while_the_caller_captures(hg):
    """Inside a capture of the caller's stream a batch with a stream of its
    own runs at once, as it does outside, and leaves the capture whole."""
    q = state(10)
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device=DEV)
    ref = batch(hg, q)
    ref.step(dt, 2)
    want = ref.get_state(0)
    b = batch(hg, q)
    b.sync()
    x = torch.zeros(8, device=DEV)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x += 1
        b.step(dt, 2)
    assert torch.equal(b.get_state(0), want)
    for k in range(1, 4):
        g.replay()
        torch.cuda.synchronize()
        assert x.tolist() == [float(k)] * 8
    assert torch.equal(b.get_state(0), want)


def test_context_on_a_stream_of_its_own(hg, busy):
    """Set, step, read and a parity hook under another current stream, with
    either side busy, inputs dropped at once and outputs read at once."""
    q = state(11)

    def march(ctx, hold):
        ctx.set_uniform_grid((0.0,) * 3, L)
        got = []
        for _ in range(3):
            hold(None)
            ctx.set_state(q * 1.0)
            torch.full_like(q, 7.0)               # takes the dropped input's memory
            ctx.step(1e-3, 2)
            hold(ctx.stream)
            got += [ctx.get_state() * 1.0, ctx.debug_face_flux(1e-3) * 1.0]
        return got

    def wait(stream):
        torch.cuda.synchronize()

    def work(stream):
        with torch.cuda.stream(stream or torch.cuda.current_stream()):
            busy()

    want = march(hg.Context(N), wait)
    for a, b in zip(march(hg.Context(N, stream=torch.cuda.Stream()), work), want):
        assert torch.equal(a, b)
