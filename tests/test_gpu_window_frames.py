"""Quantisation frames of window copies over more instances than a wave has lanes, with the
photons that reach furthest in the first, a middle and the last of them and instances without
photons: every copy's frame holds every photon's box of the copy's step, and the candidates are
those of one copy per step."""
import numpy as np
import pytest

from paper_1608_01125_amd import beams
from paper_1608_01125_amd import tril as T

from test_gpu_window import _run, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 63, 64, 65, 130])
def test_frames_hold_every_instance(torch, m):  # noqa: F811
    wl = beams.gauss_headon_1m(n=24, seed=1, w=beams.gauss_headon_1m().a.w * 3e5)
    far, parts = {0: 400.0, m // 2: -700.0, m - 1: 900.0}, ([], [])
    for k in range(m):
        for X, out in zip(beams.draw_pair(beams.gauss_headon_1m(n=24, seed=k)), parts):
            X = {f: v[:0] if k % 7 == 3 and k not in far else v for f, v in X.items()}
            X["x"] = X["x"] + far.get(k, 0.0)
            X["w"] = np.full(len(X["E"]), wl.a.w)
            out.append(X)
    (A, offA), (B, offB) = (beams.concat(p) for p in parts)
    base, cand1 = _run(wl, A, B, 150, 101, 48, 1, offA, offB)
    got, cand = _run(wl, A, B, 150, 101, 48, 32, offA, offB, dwin=16)
    assert base[3]["n_candidates"] > 0
    assert np.array_equal(cand, cand1) and got[3]["n_candidates"] == base[3]["n_candidates"]
    qa, tb = T.Beam(A, offA), T.Beam(B, offB)
    steps = 101
    ctx, pairs = T.Context(wl.dt, None, kinetic_window=32), T.Pairs(1 << 16)
    try:
        ctx.run(tb, qa, 150, steps, pairs)
        ctx.stats(pairs)
        _, frames = T.tril_dbg_quad_nodes(ctx, tb.n, steps)
    finally:
        ctx.close()
    copies = (steps + 31) // 32
    assert len(frames) == copies
    for cp in range(copies):
        first, last = 32 * cp, min(32 * cp + 31, steps - 1)
        lo, hi = frames[cp, :3], frames[cp, :3] + 65536.0 / frames[cp, 4:7]
        t = (150 + first + (last - first) // 2) * wl.dt  # the copy's step
        for a, f in enumerate(("x", "y", "z")):  # (head-on beams: no shear)
            X = B[f] + t * B["p" + f] / B["E"]
            assert lo[a] <= X.min() + 1e-3 and X.max() - 1e-3 <= hi[a]
