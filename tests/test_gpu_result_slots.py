"""Results of reductions through the pinned slots with more calls in flight
than there are slots (the rest copy)."""

import threading

import pytest
import torch

from tests.helpers import smooth_state

pytestmark = pytest.mark.gpu

N, L = (6, 5, 4), (0.6, 0.5, 0.4)


def test_more_calls_in_flight_than_slots():
    from paper_1909_01580_amd import hgks

    ctxs, want = [], []
    for k in range(80):
        ctx = hgks.Context(N)
        ctx.set_uniform_grid((0.0,) * 3, L)
        ctx.set_state(torch.tensor(smooth_state(N, L, k, mach=0.3), device="cuda:0"))
        ctxs.append(ctx)
        want.append((ctx.max_dt(0.35), ctx.totals(), ctx.check(), ctx.kinetic_energy()))
    a = torch.ones(4096, 4096, dtype=torch.float64, device="cuda:0")
    got = [None] * len(ctxs)

    def call(k):
        c = ctxs[k]
        got[k] = (c.max_dt(0.35), c.totals(), c.check(), c.kinetic_energy())

    for _ in range(2):
        for _ in range(40):
            b = a @ a                       # all the contexts' stream: every first call waits behind it
        threads = [threading.Thread(target=call, args=(k,)) for k in range(len(ctxs))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert got == want
        got[:] = [None] * len(ctxs)
    del b
