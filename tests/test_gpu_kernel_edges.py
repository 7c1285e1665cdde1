"""Sizes and states at the edges of the box kernels' dispatch: rows of the
face map around one wave's sixteen faces, supersonic interface states (the
tail branch of erfc), grids on both sides of the split reconstruction, and
more contexts than the reductions have pinned result slots.

Bars: FP64 against the oracle 1e-12 normalised (1e-10 for the flux time
derivative, a difference of near-equal terms over dt), as in the other
parity tests; the two reconstruction kernels share their per-variable code
and differ in the compiler's contraction only, a few ulp of the state."""

import numpy as np
import pytest
import torch

import oracle
from oracle import scheme
from tests.helpers import blast_state, nerr, smooth_state

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def hg():
    from paper_1909_01580_amd import hgks
    hgks.load()
    return hgks


def compare_faces(hg, n, bc, Q, L, **phys):
    prob = oracle.uniform_problem(n, (0.0,) * 3, L, bc=bc, params=oracle.Params(**phys))
    ctx = hg.Context(n, bc=bc, **phys)
    ctx.set_uniform_grid((0.0,) * 3, L)
    ctx.set_state(torch.tensor(Q, device="cuda:0"))
    dt = oracle.max_dt(prob, Q, 0.35)
    gpu = ctx.debug_face_flux(dt).cpu().numpy()
    ref = scheme.face_fluxes(prob, Q, dt)
    for k in range(2):
        err = np.abs(gpu[..., k, :] - ref[..., k, :]).max() / np.abs(ref[..., k, :]).max()
        assert err < TOL * (1 if k == 0 else 100), (k, err)
    ctx.step(dt, 2)
    e = nerr(ctx.get_state().cpu().numpy(), oracle.step(prob, Q, dt), mom_scale=True)
    assert e.max() < TOL, e


# one row of 15, 16 and 17 cells along x, rows that straddle the bands of 16
# along y, and planes whose rows along y hold sixteen faces or more
@pytest.mark.parametrize("n", [(15, 3, 2), (16, 2, 3), (17, 5, 3), (33, 17, 2), (3, 18, 16)])
@pytest.mark.parametrize("bc", ["periodic", "outflow"])
def test_face_rows(hg, n, bc):
    L = tuple(0.1 * m for m in n)
    compare_faces(hg, n, (bc,) * 3, smooth_state(n, L, 7, mach=0.5), L, mu=1e-3, prandtl=0.72)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_supersonic_stream(hg, axis, sign):
    """sqrt(lambda) |U| from 1.7 to 3.3 along one axis, subsonic along the
    others; one run per direction of the stream."""
    n, L = (9, 8, 7), (0.9, 0.8, 0.7)
    Q = smooth_state(n, L, 11, mach=0.4)
    u = sign * 3.3
    Q[4] += u * Q[1 + axis] + 0.5 * Q[0] * u * u
    Q[1 + axis] += u * Q[0]
    compare_faces(hg, n, ("periodic",) * 3, Q, L)


# 64 cells exactly, a remainder, and the last split and first unsplit sizes
@pytest.mark.parametrize("n", [(4, 4, 4), (13, 5, 2), (34, 34, 34), (35, 34, 34)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_split_reconstruction_against_batch(hg, n, precision):
    """The batch reconstructs one cell per lane at every size."""
    L = tuple(0.1 * m for m in n)
    Q = smooth_state(n, L, 3, mach=0.5)
    ctx = hg.Context(n, precision=precision)
    ctx.set_uniform_grid((0.0,) * 3, L)
    ctx.set_state(torch.tensor(Q, device="cuda:0"))
    dt = ctx.max_dt(0.35)
    ctx.step(dt, 2)
    b = hg.Batch([{"n": n, "length": L, "mu": 0.0}], precision=precision)
    b.set_state(0, torch.tensor(Q, device="cuda:0"))
    dts = torch.tensor([dt], dtype=torch.float64, device="cuda:0")  # kept while the batch's stream reads it
    torch.cuda.synchronize()
    b.step(dts, 2)
    e = nerr(ctx.get_state().cpu().numpy(), b.get_state(0).cpu().numpy())
    assert e.max() < (1e-14 if precision == "fp64" else 1e-6), e


@pytest.mark.parametrize("stencil", ["S", "S_prime"])
def test_fallback_words_repeat(hg, stencil):
    """The list of flagged cells is empty again after a step and after a
    parity hook: the words of a discontinuous state equal the oracle's at
    the first look, at a second one, and after a step was taken and undone."""
    n, L, bc = (18, 9, 7), (1.0, 1.0, 1.0), ("outflow",) * 3
    Q = blast_state(n)
    prob = oracle.uniform_problem(n, (0.0,) * 3, L, bc=bc, params=oracle.Params(stencil=stencil))
    dt = oracle.max_dt(prob, Q, 0.35)
    ref = scheme.fallback_mask(prob, Q, dt)
    assert (ref != 0).sum() > 20
    ctx = hg.Context(n, bc=bc, stencil=stencil)
    ctx.set_uniform_grid((0.0,) * 3, L)
    q = torch.tensor(Q, device="cuda:0")
    ctx.set_state(q)
    for again in range(3):
        assert np.array_equal(ctx.debug_fallback_mask(dt).cpu().numpy().astype(np.uint32), ref)
        if again == 1:
            ctx.step(dt, 2)
            ctx.set_state(q)


def test_more_contexts_than_result_slots(hg):
    """Seventy live contexts: the last few have no pinned slot and copy."""
    n, L = (6, 5, 4), (0.6, 0.5, 0.4)
    states = [smooth_state(n, L, s, mach=0.3) for s in range(70)]
    ctxs = []
    for q in states:
        ctx = hg.Context(n)
        ctx.set_uniform_grid((0.0,) * 3, L)
        ctx.set_state(torch.tensor(q, device="cuda:0"))
        ctxs.append(ctx)
    for _ in range(2):
        for q, ctx in zip(states, ctxs):
            prob = oracle.uniform_problem(n, (0.0,) * 3, L)
            ref = oracle.max_dt(prob, q, 0.35)
            assert abs(ctx.max_dt(0.35) - ref) < 1e-14 * ref
            mass = ctx.totals()[0]
            assert abs(mass - q[0].sum() * 1e-3) < 1e-13 * mass
        # slots given back serve the contexts that had none
        del ctxs[:10], states[:10]
