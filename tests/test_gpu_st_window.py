"""Windows of the cloud traversal (32 steps per descent, 8 queries per wave): cuts of the
first and the last window, query counts about the wave's, instances of one row and none, a
launch limited to a few steps, crossing beams; every bin-pair yield against the oracle."""
import numpy as np
import pytest

from oracle import st_oracle as SO
from paper_1608_01125_amd import beams
from paper_1608_01125_amd import tril as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a GPU"
    return _t


def _table(torch, A, B, ga, gb, wl, k0, n_steps, offA=None, offB=None, step_batch=0):
    sides = []
    for beam, g, off in ((A, ga, offA), (B, gb, offB)):
        b = T.Beam(beam, off)
        bins = torch.empty(max(b.n, 1), dtype=torch.int32, device="cuda")
        T.tril_st_bin(b, g, bins)
        sides.append((b, bins))
    (qa, qb), (tb, tbins) = sides
    ctx = T.Context(wl.dt, None, step_batch=step_batch)
    tab = T.StTable(18)
    try:
        tot = T.tril_st_exact(ctx, tb, tbins, gb.n_bins, qa, qb, ga.cell, k0, n_steps, tab)
    finally:
        ctx.close()
    keys, ys = tab.items()
    return keys, ys, tot


def _reference(A, B, ga, gb, wl, k0, n_steps, offA, offB):
    ba, _ = SO.bin_beam(A, ga)
    bb, _ = SO.bin_beam(B, gb)
    tab, tot = {}, 0.0
    for m in range(len(offA) - 1):
        a, b = slice(offA[m], offA[m + 1]), slice(offB[m], offB[m + 1])
        if offA[m] == offA[m + 1] or offB[m] == offB[m + 1]:
            continue
        t, s = SO.st_table({k: v[a] for k, v in A.items()}, ba[a],
                           {k: v[b] for k, v in B.items()}, bb[b], gb.n_bins, wl.dt, k0, n_steps,
                           ga.cell)
        for k, v in t.items():
            tab[k] = tab.get(k, 0.0) + v
        tot += s
    return tab, tot


def _check(got, ref):
    (keys, ys, tot), (tab, ref_tot) = got, ref
    rk = np.array(sorted(tab), dtype=np.int64)
    assert np.array_equal(keys, rk)
    np.testing.assert_allclose(ys, np.array([tab[k] for k in rk]), rtol=1e-9, atol=0)
    assert abs(tot - ref_tot) <= 1e-9 * max(ref_tot, 1e-300)


@pytest.mark.parametrize("k0,n_steps,step_batch", [
    (200, 1, 0), (192, 32, 0), (191, 33, 0), (185, 40, 0), (190, 33, 5), (190, 20, 1), (200, 0, 0)])
@pytest.mark.parametrize("n", [1, 7, 9, 65])
def test_windows_and_query_counts(torch, n, k0, n_steps, step_batch):
    wl = beams.st_headon(4000, seed=5)
    A, B = beams.draw_pair(wl)
    ga, gb = beams.st_grid(wl, "a", A), beams.st_grid(wl, "b", B)
    core = np.argsort(A["x"] ** 2 + A["y"] ** 2 + (0.2 * (A["z"] + 20.0)) ** 2)[:n]
    A = {k: np.ascontiguousarray(v[core]) for k, v in A.items()}
    got = _table(torch, A, B, ga, gb, wl, k0, n_steps, step_batch=step_batch)
    ref = _reference(A, B, ga, gb, wl, k0, n_steps, [0, n], [0, 4000])
    if n > 1 and n_steps > 10:
        assert ref[1] > 0
    _check(got, ref)


@pytest.mark.parametrize("sizes", [((1, 0, 33, 1), (1, 40, 1, 700)), ((40, 3, 2, 5), (600, 1, 1, 300)),
                                   ((7,) * 20, (90,) * 20)])
def test_instances_share_waves(torch, sizes):
    """Waves whose queries belong to several instances, some of one row or empty."""
    wl = beams.st_train_instance(3, 4000)
    A, B = beams.draw_pair(wl)
    ga, gb = beams.st_grid(wl, "a", A), beams.st_grid(wl, "b", B)
    offA, offB = (np.concatenate([[0], np.cumsum(s)]).astype(np.int64) for s in sizes)
    t = 0.5 * wl.n_steps * wl.dt
    rows = [np.argsort(sum((b[k] + t * b["p" + k] / b["E"]) ** 2 for k in "xyz"))[: o[-1]]
            for b, o in ((A, offA), (B, offB))]
    A, B = ({k: np.ascontiguousarray(v[r]) for k, v in b.items()} for b, r in zip((A, B), rows))
    got = _table(torch, A, B, ga, gb, wl, 150, 100, offA, offB)
    ref = _reference(A, B, ga, gb, wl, 150, 100, offA, offB)
    assert ref[1] > 0
    _check(got, ref)
