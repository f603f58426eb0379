"""What a statistical pass leaves in the context: its hierarchies are of clouds over windows of
steps, which tril_collide does not take for a step's build, whatever their number."""
import numpy as np
import pytest

from paper_1608_01125_amd import beams
from paper_1608_01125_amd import tril as T

from test_gpu_st_window import torch  # noqa: F401

pytestmark = pytest.mark.gpu
N = 1500


def _setup(torch):  # noqa: F811
    wl = beams.st_headon(N, seed=4)
    A, B = beams.draw_pair(wl)
    A["w"][:], B["w"][:] = 3e15, 3e15  # some collide in every middle step
    ga, gb = beams.st_grid(wl, "a", A), beams.st_grid(wl, "b", B)
    sides = []
    for b, g in ((A, ga), (B, gb)):
        dev = T.Beam(b)
        bins = torch.empty(N, dtype=torch.int32, device="cuda")
        T.tril_st_bin(dev, g, bins)
        sides.append((dev, bins))
    return wl, ga, gb, sides


def _hits(ctx, query, step):
    pairs = T.Pairs(1 << 16)
    ctx.collide(query, step, pairs)
    return sorted(zip(*(v.tolist() for v in pairs.numpy())))


@pytest.mark.parametrize("flags", [0, 0x10])  # hierarchy, grid
@pytest.mark.parametrize("k0,n_steps", [(200, 1), (0, 20), (200, 20), (0, 32), (192, 32), (150, 100),
                                        (200, 0)])
def test_collide_needs_a_build_of_its_own(torch, k0, n_steps, flags):  # noqa: F811
    wl, ga, gb, ((qa, qbins), (tb, tbins)) = _setup(torch)
    last = k0 + max(n_steps, 1) - 1
    ctx = T.Context(wl.dt, None, flags=flags)
    try:
        ctx.build(tb, last)
        want = _hits(ctx, qa, last)
        for swarm in (False, True):
            if swarm:
                T.tril_ip_swarm(ctx, tb, tbins, gb.n_bins, qa, qbins, (1e-3,) * 3, k0, n_steps,
                                T.StTable(12), T.StTable(12))
            else:
                T.tril_st_exact(ctx, tb, tbins, gb.n_bins, qa, qbins, ga.cell, k0, n_steps,
                                T.StTable(18))
            for step in {last, k0, 0}:
                with pytest.raises(T.TrilError) as ei:
                    ctx.collide(qa, step, T.Pairs(16))
                assert ei.value.code == T.TRIL_E_STATE
            ctx.build(tb, last)
            assert _hits(ctx, qa, last) == want
        if last >= 190:
            assert want
    finally:
        ctx.close()


@pytest.mark.parametrize("k0,n_steps", [(192, 32), (200, 1), (70, 20), (185, 40), (100, 100)])
def test_boxes_of_a_pass_hold_its_clouds(torch, k0, n_steps):  # noqa: F811
    """tril_dbg_boxes after a pass gives its last launch's windows, of 32 steps (or of the whole
    pass, where that is shorter): the clouds of every mid-step, and no more than a step beyond."""
    wl, ga, gb, ((qa, qbins), (tb, tbins)) = _setup(torch)
    B = beams.draw_pair(wl)[1]
    win = min(32, n_steps)
    ctx = T.Context(wl.dt, None)
    try:
        T.tril_st_exact(ctx, tb, tbins, gb.n_bins, qa, qbins, ga.cell, k0, n_steps, T.StTable(18))
        box = T.tril_dbg_boxes(ctx, 0, (n_steps // win) * N)
    finally:
        ctx.close()
    windows = len(box["lo"]) // N
    assert windows >= 1 and len(box["lo"]) == windows * N
    for s in range(windows):
        first = ((k0 + n_steps - 1) // win - windows + 1 + s) * win
        rows = slice(s * N, (s + 1) * N)
        for a, f in enumerate(("x", "y", "z")):
            mid = [B[f] + (first + t + 0.5) * wl.dt * B["p" + f] / B["E"] for t in (0, win - 1)]
            lo, hi = np.minimum(*mid) - 0.5 * ga.cell[a], np.maximum(*mid) + 0.5 * ga.cell[a]
            assert (box["lo"][rows, a] <= lo).all() and (box["hi"][rows, a] >= hi).all()
            assert (box["lo"][rows, a] > lo - wl.dt).all() and (box["hi"][rows, a] < hi + wl.dt).all()
