"""Cloud traversals of more waves than one grid holds (eight threads per query and window, at most
2^32 - 1 a grid): 2^20 macro-particles over 512 windows of one step, as the swarms' pair finding
has them, in one batch of steps and in batches of 64."""
import numpy as np
import pytest

from paper_1608_01125_amd import tril as T

from test_gpu_swarm import torch  # noqa: F401

pytestmark = pytest.mark.gpu

N, TARGETS, STEPS, DT, CELL = 1 << 20, 40, 512, 0.1, (0.05, 0.05, 0.05)


def _beam(n, seed, side, sign):
    rng = np.random.default_rng(seed)
    b = {f: rng.uniform(-side, side, n) for f in ("x", "y")}
    b["z"] = -sign * rng.uniform(1.0, 50.0, n)
    b["px"], b["py"], b["pz"] = np.zeros(n), np.zeros(n), np.full(n, 2.0 * sign)
    b["E"], b["w"] = np.full(n, 2.0), np.ones(n)
    return b


def test_more_waves_than_a_grid_holds(torch):  # noqa: F811
    A, B = _beam(N, 1, 50.0, 1.0), _beam(TARGETS, 2, 49.0, -1.0)
    qa, tb = T.Beam(A), T.Beam(B)
    qbins = torch.zeros(N, dtype=torch.int32, device="cuda")
    tbins = torch.zeros(TARGETS, dtype=torch.int32, device="cuda")
    found = []
    for step_batch in (0, 64):
        ctx = T.Context(DT, None, step_batch=step_batch)
        pt, tab = T.StTable(12), T.StTable(4)
        try:
            T.tril_ip_swarm(ctx, tb, tbins, 1, qa, qbins, CELL, 0, STEPS, pt, tab)
        finally:
            ctx.close()
        found.append(pt.items())
    assert np.array_equal(found[0][0], found[1][0])
    assert np.array_equal(found[0][1], found[1][1])
    # pairs that meet for certain: inside the cells' edges across, and within the run along
    meet = []
    for j in range(TARGETS):
        dx, dy = np.abs(A["x"] - B["x"][j]), np.abs(A["y"] - B["y"][j])
        for i in np.nonzero(np.maximum(dx, dy) < 0.99 * CELL[0])[0]:
            at = 0.5 * (B["z"][j] - A["z"][i])
            if 0.1 < at < STEPS * DT - 0.1:
                meet.append((at, int(i) * TARGETS + j))
    assert len(meet) > 20 and min(meet)[0] < 15.0 and max(meet)[0] > 35.0
    assert {k for _, k in meet} <= set(found[0][0].tolist())


def test_more_waves_of_fast_clouds(torch):  # noqa: F811
    """The same of the cloud traversal, steps of eight cells (windows of one step)."""
    A, B = _beam(N, 3, 50.0, 1.0), _beam(TARGETS, 4, 49.0, -1.0)
    for b in (A, B):
        b["z"] *= 4.0
    qa, tb = T.Beam(A), T.Beam(B)
    qbins = torch.arange(N, dtype=torch.int32, device="cuda")
    tbins = torch.arange(TARGETS, dtype=torch.int32, device="cuda")
    found = []
    for step_batch in (0, 64):
        ctx, tab = T.Context(4 * DT, None, step_batch=step_batch), T.StTable(12)
        try:
            tot = T.tril_st_exact(ctx, tb, tbins, TARGETS, qa, qbins, CELL, 0, STEPS, tab)
        finally:
            ctx.close()
        found.append((*tab.items(), tot))
    assert len(found[0][0]) > 2 and np.array_equal(found[0][0], found[1][0])
    # a key's value is one sum over a pair's steps, the total one over all of them
    np.testing.assert_allclose(found[0][1], found[1][1], rtol=1e-14, atol=0)
    assert found[0][2] == pytest.approx(found[1][2], rel=1e-12)
