"""Runs whose beams cross at an angle descend forms in sheared coordinates: the candidates (the
last launch's, as a multiset, and the count over the run), hits and pairs must be those of one
copy of the hierarchy per step, which no shear enters."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1608_01125_amd import beams

from test_gpu_window import _run, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _crossing(phis, n=2500, boost=3e3, shift=None, opening=0.010):
    parts = []
    for k, phi in enumerate(phis):
        wl = beams.gauss_headon_1m(n=n - 300 * k, seed=3 + k)
        wl = beams.gauss_headon_1m(n=n - 300 * k, seed=3 + k, w=wl.a.w * boost)
        wl = replace(wl, a=replace(wl.a, opening=opening),
                     b=replace(wl.b, phi_deg=phi, opening=opening))
        parts.append(beams.draw_pair(wl))
    A, offA = beams.concat([p[0] for p in parts])
    B, offB = beams.concat([p[1] for p in parts])
    if shift is not None:
        for X in (A, B):
            for a, f in enumerate(("x", "y", "z")):
                X[f] = X[f] + shift[a]
    if len(phis) == 1:
        offA = offB = None
    return wl, A, B, offA, offB


@pytest.mark.parametrize("phis,win,dwin,shift,opening", [
    ((150.0,), 32, 8, None, 0.010), ((150.0,), 16, 3, None, 0.010), ((90.0,), 32, 32, None, 0.010),
    ((90.0,), 16, 2, None, 0.010), ((35.0,), 32, 16, None, 0.010), ((120.0,), 32, 8, None, 0.6),
    ((150.0, 90.0, 180.0, 100.0), 32, 8, None, 0.010),
    ((110.0,), 16, 16, (1000.0, -700.0, 900.0), 0.010)])
def test_candidates_equal_per_step_copies(torch, phis, win, dwin, shift, opening):  # noqa: F811
    wl, A, B, offA, offB = _crossing(phis, boost=3e4 if shift else 3e3, shift=shift,
                                     opening=opening)
    base, cand1 = _run(wl, A, B, 150, 101, 48, 1, offA, offB)
    assert base[3]["n_candidates"] > 20
    got, cand = _run(wl, A, B, 150, 101, 48, win, offA, offB, dwin=dwin)
    assert np.array_equal(cand, cand1)
    for f in ("n_candidates", "n_hits", "n_pairs", "n_queries"):
        assert got[3][f] == base[3][f]
    for a, b in zip(got[:3], base[:3]):
        assert np.array_equal(a, b)
