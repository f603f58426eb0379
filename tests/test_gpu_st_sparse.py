"""Clouds much smaller than their spacing, alone or beside a dense core: waves whose queries'
boxes fill little of their hull test the nodes against each box, the others against the hull;
every bin-pair yield against the oracle, one instance and several in a wave."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1608_01125_amd import beams

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
