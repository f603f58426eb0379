"""Clouds much smaller than their spacing, alone or beside a dense core: waves whose queries'
boxes fill little of their hull test the nodes against each box, the others against the hull;
every bin-pair yield against the oracle, one instance and several in a wave."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1608_01125_amd import beams
from paper_1608_01125_amd import tril as T

from test_gpu_st_window import _check, _reference, _table, torch  # noqa: F401

pytestmark = pytest.mark.gpu
N = 3000


def _beams(core, phi):
    wl = beams.st_headon(N, seed=12)
    wl = replace(wl, b=replace(wl.b, phi_deg=phi))
    A, B = beams.draw_pair(wl)
    t = 0.5 * wl.n_steps * wl.dt
    for X in (A, B):  # pulled together about where both centres meet, at that time
        for f in "xyz":
            u = X["p" + f] / X["E"]
            at = X[f] + t * u
            at[:core] *= 0.05
            X[f] = at - t * u
    grids = [replace(beams.st_grid(wl, w, X), n_pos=(160, 160, 160), n_e=1, n_th=1)
             for w, X in (("a", A), ("b", B))]
    return wl, A, B, grids


@pytest.mark.parametrize("phi", [180.0, 90.0])
@pytest.mark.parametrize("core", [0, 400])
@pytest.mark.parametrize("k0,n_steps,step_batch", [(170, 60, 0), (170, 60, 1), (199, 1, 0)])
@pytest.mark.parametrize("inst", [1, 7])
def test_sparse_clouds(torch, core, phi, k0, n_steps, step_batch, inst):  # noqa: F811
    wl, A, B, (ga, gb) = _beams(core, phi)
    offA = offB = None
    if inst > 1:
        offA = np.linspace(0, N, inst + 1).astype(np.int64)
        offB = np.minimum(offA + 5, N)
        offB[0] = 0
    got = _table(torch, A, B, ga, gb, wl, k0, n_steps, offA, offB, step_batch=step_batch)
    one = np.array([0, N])
    ref = _reference(A, B, ga, gb, wl, k0, n_steps, one if offA is None else offA,
                     one if offB is None else offB)
    if n_steps > 1 and inst == 1:
        assert len(ref[0]) > 30
    _check(got, ref)


@pytest.mark.parametrize("phi", [180.0, 90.0])
@pytest.mark.parametrize("inst", [1, 5])
def test_steps_of_many_edges(torch, phi, inst):  # noqa: F811
    """Sparse clouds that move 40 edges per step take a lane per query and step, in launches of one
    step (375 waves) the shared descent: yields against the oracle, and depleted yields per cloud
    pair the same by both."""
    wl, A, B, (ga, gb) = _beams(400, phi)
    wl = replace(wl, dt=4.0, n_steps=60)
    offA = offB = None
    if inst > 1:  # one without targets, one of a single target
        offA = np.array([0, 900, 901, 1500, 2200, N])
        offB = np.array([0, 900, 1500, 1500, 1501, N])
    one = np.array([0, N])
    ref = _reference(A, B, ga, gb, wl, 0, 60, one if offA is None else offA,
                     one if offB is None else offB)
    assert len(ref[0]) > 30
    for step_batch in (0, 1):
        _check(_table(torch, A, B, ga, gb, wl, 0, 60, offA, offB, step_batch=step_batch), ref)
    sides = []
    for X, g, off in ((A, ga, offA), (B, gb, offB)):
        b, bins = T.Beam(X, off), torch.empty(N, dtype=torch.int32, device="cuda")
        T.tril_st_bin(b, g, bins)
        sides.append((b, bins))
    got = []
    for step_batch in (0, 1):
        ctx, tab, pt = T.Context(wl.dt, None, step_batch=step_batch), T.StTable(18), T.StTable(18)
        try:
            tot = T.tril_st_exact_depleted(ctx, *sides[1], gb.n_bins, *sides[0], ga.cell, 0, 60, pt, tab)
        finally:
            ctx.close()
        got.append((*pt.items(), *tab.items(), tot))
    assert len(got[0][0]) > 30
    for a, b in zip(got[0][:4:2], got[1][:4:2]):
        assert np.array_equal(a, b)
    for a, b in zip(got[0][1:4:2], got[1][1:4:2]):
        np.testing.assert_allclose(a, b, rtol=1e-12, atol=0)
    assert got[0][4] == pytest.approx(got[1][4], rel=1e-12)
