"""Steps over the range of the nonlinear weights, through every kernel that
forms them: any positive epsilon is a configuration, and data in any units.

* Scale: with the state times 2^300 (2e90) and epsilon times 2^600 every
  product of the scheme is the unscaled one times a power of two, so the step
  must return the unscaled step's bits times 2^300 (indicators of 1e180; the
  unscaled side runs at an epsilon of 2e-189).  Where values themselves are
  far below the data (the relaxation factor leaves 1e-200 in a momentum at
  rest) a product may leave the format on one side only: up to 2^-500.
* Epsilon 1e-200 on a state that is uniform over most of the grid, where
  every indicator there is the bare epsilon, against the oracle: 1e-12
  normalised, the bar of the other parity tests."""

import numpy as np
import pytest
import torch

import oracle
from paper_1909_01580_amd import workloads as wl
from tests.helpers import blast_state, nerr

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
L = (1.0, 1.0, 1.0)
# below and above the size up to which the reconstruction splits a cell's variables over waves
SIZES = [(14, 11, 9), (36, 34, 33)]
OPTIONS = {"S": {}, "S_prime": {"stencil": "S_prime"}, "characteristic": {"characteristic": True}}


@pytest.fixture(scope="module")
def hg():
    from paper_1909_01580_amd import hgks
    hgks.load()
    return hgks


def step_box(hg, n, Q, **kw):
    ctx = hg.Context(n, bc=("outflow",) * 3, **kw)
    ctx.set_uniform_grid((0.0,) * 3, L)
    ctx.set_state(torch.tensor(Q, device=DEV))
    dt = ctx.max_dt(0.35)
    ctx.step(dt, 2)
    return dt, ctx.get_state().cpu().numpy()


def step_batch(hg, n, Q, **kw):
    kw["characteristic"] = int(kw.get("characteristic", False))
    b = hg.Batch([{"n": n, "length": L, "mu": 0.0}], precision="fp64", **kw)
    b.set_state(0, torch.tensor(Q, device=DEV))
    dt = torch.empty(1, dtype=torch.float64, device=DEV)
    b.max_dt(0.35, dt)
    b.step(dt, 2)
    return float(dt), b.get_state(0).cpu().numpy()


def step_hex(hg, n, Q, **kw):
    ctx = hg.Context(n, moving=True, **kw)
    ctx.set_vertices(torch.tensor(wl.sine_mesh_vertices(n, 0.0, amp=0.1, static=True), device=DEV), (2.0,) * 3)
    ctx.set_state(torch.tensor(Q, device=DEV))
    dt = ctx.max_dt(0.35)
    ctx.step(dt, 2)
    return dt, ctx.get_state().cpu().numpy()


@pytest.mark.parametrize("step", [step_box, step_batch, step_hex])
@pytest.mark.parametrize("option", list(OPTIONS))
@pytest.mark.parametrize("n", SIZES)
def test_scale_of_the_data(hg, step, option, n):
    Q = blast_state(n)
    dt0, ref = step(hg, n, Q, weno_eps=2.0 ** -627, **OPTIONS[option])
    dt1, out = step(hg, n, Q * 2.0 ** 300, weno_eps=2.0 ** -27, **OPTIONS[option])
    assert np.isfinite(ref).all() and np.abs(ref - Q).max() > 1e-3
    assert dt0 == dt1
    assert np.abs(out * 2.0 ** -300 - ref).max() <= 2.0 ** -500


@pytest.mark.parametrize("option", list(OPTIONS))
@pytest.mark.parametrize("n", SIZES)
def test_bare_epsilon(hg, option, n):
    """The larger size on a thin slice of the oracle's work: a uniform state stays as it is."""
    kw = dict(weno_eps=1e-200, **OPTIONS[option])
    uniform = wl.conservative(*[np.full(n[::-1], x) for x in (1.2, 0.3, -0.2, 0.1, 0.8)])
    dt, out = step_box(hg, n, uniform, **kw)
    assert nerr(out, uniform).max() < 1e-14
    _, out = step_batch(hg, n, uniform, **kw)
    assert nerr(out, uniform).max() < 1e-14
    if n != SIZES[0]:
        return
    Q = blast_state(n)
    prob = oracle.uniform_problem(n, (0.0,) * 3, L, bc=("outflow",) * 3, params=oracle.Params(**kw))
    dt, out = step_box(hg, n, Q, **kw)
    assert abs(dt - oracle.max_dt(prob, Q, 0.35)) < 1e-14 * dt
    assert nerr(out, oracle.step(prob, Q, dt), mom_scale=True).max() < 1e-12
