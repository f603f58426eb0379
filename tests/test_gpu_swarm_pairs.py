"""Pair finding of the swarms: one key per macro-particle pair of an instance whose clouds, swept
over some step, meet above threshold. The boxes are single precision, rounded outward and padded
by the collision radius (below 1e-8 um), so pairs whose FP64 boxes overlap by 1e-5 um (positions
below 32 um round by at most 2e-6) have to be there and pairs that are 1e-5 um apart must not."""
import numpy as np
import pytest

from paper_1608_01125_amd import tril as T

from test_gpu_swarm import ME, _check, _run, _tiny, torch  # noqa: F401

pytestmark = pytest.mark.gpu
CELL, DT, K0, STEPS, MARGIN = (0.4, 0.6, 0.5), 0.25, 3, 37, 1e-5


def _beam(n, seed, sign):
    rng = np.random.default_rng(seed)
    b = {f: rng.normal(0.0, 3.0, n) for f in ("x", "y")}
    b["z"] = -sign * rng.uniform(0.0, 12.0, n)
    d = np.stack([rng.normal(0, 0.3, n), rng.normal(0, 0.3, n), np.full(n, sign)], 1)
    d /= np.linalg.norm(d, axis=1)[:, None]
    b["E"] = rng.uniform(0.3, 1.2, n)
    for a, f in enumerate(("px", "py", "pz")):
        b[f] = b["E"] * d[:, a]
    b["w"] = np.ones(n)
    return b


def _meet(A, B, offA, offB, margin):
    """Keys of the pairs whose swept boxes overlap by more than -margin in some step."""
    nB, keys = len(B["E"]), set()
    for m in range(len(offA) - 1):
        i, j = np.arange(offA[m], offA[m + 1])[:, None], np.arange(offB[m], offB[m + 1])[None]
        cphi = sum((A[p][i] / A["E"][i]) * (B[p][j] / B["E"][j]) for p in ("px", "py", "pz"))
        above = A["E"][i] * B["E"][j] * (1.0 - cphi) / (2.0 * ME * ME) > 1.0
        met = np.zeros(above.shape, bool)
        for k in range(K0, K0 + STEPS):
            ok = above.copy()
            for a, f in enumerate(("x", "y", "z")):
                e = [(X[f] + k * DT * X["p" + f] / X["E"], X[f] + (k + 1) * DT * X["p" + f] / X["E"])
                     for X in (A, B)]
                lo, hi = [np.minimum(*v) for v in e], [np.maximum(*v) for v in e]
                ok &= (lo[0][i] - hi[1][j] < CELL[a] + margin) & (lo[1][j] - hi[0][i] < CELL[a] + margin)
            met |= ok
        ii, jj = np.nonzero(met)
        keys |= set(((ii + offA[m]) * nB + jj + offB[m]).tolist())
    return keys


@pytest.mark.parametrize("step_batch", [0, 1, 5])
@pytest.mark.parametrize("sizes", [((1,), (1,)), ((63,), (300,)), ((257,), (129,)),
                                   ((1, 0, 33, 1, 70), (1, 40, 1, 300, 90)), ((40, 5), (0, 1)),
                                   ((900, 0, 1, 40), (200, 40, 300, 1))])  # one lane a query
def test_pairs_whose_swept_clouds_meet(torch, sizes, step_batch):  # noqa: F811
    offA, offB = (np.concatenate([[0], np.cumsum(s)]).astype(np.int64) for s in sizes)
    A, B = _beam(int(offA[-1]), 5, 1.0), _beam(int(offB[-1]), 6, -1.0)
    if sizes[0] == (1,):
        for f in ("x", "y"):
            B[f][:] = A[f]
        for b, sign in ((A, 1.0), (B, -1.0)):
            b["px"][:], b["py"][:], b["pz"][:] = 0.0, 0.0, sign * b["E"]
        B["E"][:], B["pz"][:] = 2.0, -2.0
    sides = []
    for b, off in ((A, offA), (B, offB)):
        n = len(b["E"])
        sides.append((T.Beam(b, off), torch.zeros(n, dtype=torch.int32, device="cuda")))
    ctx = T.Context(DT, None, step_batch=step_batch)
    pt, tab = T.StTable(16), T.StTable(4)
    try:
        T.tril_ip_swarm(ctx, *sides[1], 1, *sides[0], CELL, K0, STEPS, pt, tab)
    finally:
        ctx.close()
    got = set(pt.items()[0].tolist())
    sure, may = _meet(A, B, offA, offB, -MARGIN), _meet(A, B, offA, offB, MARGIN)
    if sizes != ((40, 5), (0, 1)):
        assert sure
    assert sure <= got <= may


@pytest.mark.parametrize("pair_log2", [0, 5, 6, 9, 25])
def test_pairs_are_found_in_tables_of_any_size(torch, pair_log2):  # noqa: F811
    """The table's pairs are listed before they are counted, those of one block of 64 photons
    apart from the others, and tables above 2^24 slots in pieces: one pair in one slot, full
    words, and two pieces."""
    n = 1 if pair_log2 == 0 else 6
    A, B = _tiny(31, n, along=1e-3, spread=1e-9)
    A["w"] = np.resize([64.0, 65.0, 1.0, 600.0, 63.0, 513.0], n)
    B["w"] = np.resize([500.0, 3.0, 64.0, 65.0, 1.0], n)
    if pair_log2 == 5:  # 30 pairs of 32 slots
        B = {f: v[:5] for f, v in B.items()}
    _check(torch, A, B, (4e-9,) * 3, pair_log2=pair_log2)


@pytest.mark.parametrize("ni,nj", [(132334651, 1073072517), (132334651, 1065067422), (70001, 65537)])
def test_counts_of_the_largest_swarms(torch, ni, nj):  # noqa: F811
    """Clouds far smaller than r that pass through each other: every real pair collides. The
    pair's count is the whole number rounded once, also above 2^53, where a sum of its parts in
    double precision rounds to a neighbour in any order (the first two)."""
    A, B = _tiny(41, 1, spread=0.0, along=0.0)
    A["w"][0], B["w"][0] = ni, nj
    for _ in range(3):
        tot, pk, pv, bk, bv = _run(torch, A, B, (1e-11,) * 3)
        assert tot == ni * nj
        assert pk.tolist() == bk.tolist() == [0] and pv[0] == bv[0] == float(ni * nj)
