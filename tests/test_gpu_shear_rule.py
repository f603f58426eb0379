"""Which runs shear their node boxes: those whose descents cover more along the relative motion
than the target's nodes are wide. Dense beams do (candidates those of one copy per step, with
descents of 3 to 32 steps, wide openings, several instances of which some shear and some do not,
coordinates of 1e3 um), sparse ones and wide ones with short descents do not. Whether the forms
are sheared shows in their frames: with the nodes kept for inspection they never are."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1608_01125_amd import beams
from paper_1608_01125_amd import tril as T

from test_gpu_window import _run, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _beams(phis, sizes, n=2500, opening=0.010, shift=None):
    parts = []
    for k, (phi, size) in enumerate(zip(phis, sizes)):
        wl = beams.gauss_headon_1m(n=n - 300 * k, seed=3 + k)
        wl = beams.gauss_headon_1m(n=n - 300 * k, seed=3 + k, w=wl.a.w * 3e2)
        a = replace(wl.a, size_r=size, size_z=2 * size, opening=opening)
        wl = replace(wl, a=a, b=replace(a, phi_deg=phi))
        parts.append(beams.draw_pair(wl))
    A, offA = beams.concat([p[0] for p in parts])
    B, offB = beams.concat([p[1] for p in parts])
    if shift is not None:
        for X in (A, B):
            for a, f in enumerate(("x", "y", "z")):
                X[f] = X[f] + shift[a]
    return wl, A, B, (None, None) if len(phis) == 1 else (offA, offB)


def _sheared(wl, A, B, offs, win, dwin):
    """Do the copies' frames differ from those of unsheared forms?"""
    frames = []
    for keep in (False, True):
        ctx = T.Context(wl.dt, None, kinetic_window=win, descent_window=dwin)
        try:
            T.tril_dbg_keep_nodes(ctx, keep)
            pairs, tb = T.Pairs(1 << 18), T.Beam(B, offs[1])
            ctx.run(tb, T.Beam(A, offs[0]), 150, 101, pairs)
            frames.append(T.tril_dbg_quad_nodes(ctx, tb.n, 101)[1])
        finally:
            ctx.close()
    return not np.array_equal(frames[0], frames[1])


@pytest.mark.parametrize("phis,sizes,win,dwin,opening,shift,sheared", [
    ((150.0,), (0.3,), 32, 8, 0.010, None, True), ((150.0,), (0.3,), 16, 3, 0.010, None, True),
    ((150.0,), (0.3,), 16, 2, 0.010, None, False), ((90.0,), (0.3,), 32, 32, 0.010, None, True),
    ((35.0,), (0.1,), 32, 16, 0.010, None, True), ((120.0,), (0.1,), 32, 8, 0.6, None, True),
    ((120.0,), (2.0,), 32, 4, 0.6, None, False), ((90.0,), (8.0,), 32, 4, 0.010, None, False),
    ((150.0, 90.0, 180.0, 100.0), (0.2, 6.0, 0.2, 0.3), 32, 8, 0.010, None, None),
    ((180.0,), (0.1,), 32, 16, 0.0, None, False),
    ((110.0,), (0.3,), 16, 16, 0.010, (1000.0, -700.0, 900.0), True)])
def test_candidates_and_rule(torch, phis, sizes, win, dwin, opening, shift, sheared):  # noqa: F811
    wl, A, B, offs = _beams(phis, sizes, opening=opening, shift=shift)
    base, cand1 = _run(wl, A, B, 150, 101, 48, 1, *offs)
    got, cand = _run(wl, A, B, 150, 101, 48, win, *offs, dwin=dwin)
    if max(sizes) < 1.0:
        assert base[3]["n_candidates"] > 20
    assert np.array_equal(cand, cand1)
    for f in ("n_candidates", "n_hits", "n_pairs", "n_queries"):
        assert got[3][f] == base[3][f]
    for a, b in zip(got[:3], base[:3]):
        assert np.array_equal(a, b)
    if sheared is not None:  # (a frame of all instances is that of the widest, unsheared)
        assert _sheared(wl, A, B, offs, win, dwin) == sheared
