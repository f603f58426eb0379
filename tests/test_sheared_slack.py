"""The slack of the hull over sheared node boxes where rounding decides (host check, no GPU).

A leaf's box touches the query's at one step of the descent, on every axis, at the corner where
the two also touch in the sheared coordinates, as closely as FP32 lets two moved boxes touch.
Coordinates reach 1e5 um on one axis and 1e-3 on another, directions are an instance of one
photon's, and the shear's factors lie near +-1. Every such leaf's sheared box at the copy's step
has to be inside the hull, also with half the slack (the bound beside wslack claims that half is
to spare); without the slack, and without the part |a_i| wslack_k of the sheared axis alone, some
are outside, so the check has teeth."""
import numpy as np

from test_descent_bounds import F, exact_hits, moved_axis, wslack
from test_sheared_bounds import _shear


def _touching(n, seed):
    """Records that touch at step `meet` on every axis, the shear (a, k), steps and the copy's r."""
    rng = np.random.default_rng(seed)
    rows = np.arange(n)[:, None]
    k = rng.integers(0, 3, size=(n, 1))
    a = (rng.choice([-1.0, 1.0], size=(n, 3)) * rng.choice([1.0, 0.999, 0.7, 0.1], size=(n, 3))).astype(F)
    a[rows, k] = 0.0
    side_k = rng.choice([-1.0, 1.0], size=(n, 1))
    # the corner that stays a corner: along a_i > 0 the target lies on opposite sides of i and k
    side = np.where(a == 0, side_k, -np.sign(a) * side_k)

    def mag():
        return 10.0 ** rng.uniform(-3, 5, size=(n, 3)) * rng.choice([-1.0, 1.0], size=(n, 3))

    ql = mag().astype(F)
    qd, td = ((rng.uniform(0.01, 0.1, size=(n, 3)) * rng.choice([-1.0, 1.0], size=(n, 3))).astype(F)
              for _ in range(2))
    qw, tw = ((10.0 ** rng.uniform(-4, -1, size=(n, 3))).astype(F) for _ in range(2))
    s0 = rng.integers(0, 32, size=(n, 1))
    ln = rng.integers(1, 33, size=(n, 1))
    meet = (s0 + rng.integers(0, 32, size=(n, 1)) % ln).astype(F)
    q_lo, q_hi = moved_axis(ql, qd, qw, meet)
    tl = (ql.astype(np.float64) + meet * (qd.astype(np.float64) - td)).astype(F)
    for _ in range(12):  # closer until the FP32 boxes touch or stop moving
        t_lo, t_hi = moved_axis(tl, td, tw, meet)
        gap = np.where(side > 0, t_lo.astype(np.float64) - q_hi, q_lo.astype(np.float64) - t_hi)
        tl = (tl.astype(np.float64) - side * gap).astype(F)
    for _ in range(4):  # a step too far apart: one FP32 step back
        t_lo, t_hi = moved_axis(tl, td, tw, meet)
        apart = np.where(side > 0, t_lo > q_hi, t_hi < q_lo)
        tl = np.where(apart, np.nextafter(tl, np.where(side > 0, F(-np.inf), F(np.inf))), tl).astype(F)
    r = (s0 // 32) * 32 + rng.integers(0, 32, size=(n, 1))
    return (ql, qd, qw), (tl, td, tw), s0, ln, a, k, r


def _outside(slack, along=1.0, n=80_000, seed=7):
    """Leaves that meet the query, and those of them outside the hull; along: the share of the
    sheared axis's part of the slack."""
    q, t, s0, ln, a, k, r = _touching(n, seed)
    (ql, qd, qw), (tl, td, tw) = q, t
    rows = np.arange(n)[:, None]
    vlo, vhi = np.nextafter(td, F(-np.inf)), np.nextafter(td, F(np.inf))
    e = a.astype(np.float64) * vlo[rows, k]
    f = a.astype(np.float64) * vhi[rows, k]
    glo = np.where(a != 0, np.nextafter((vlo - np.fmax(e, f)).astype(F), F(-np.inf)), vlo)
    ghi = np.where(a != 0, np.nextafter((vhi - np.fmin(e, f)).astype(F), F(np.inf)), vhi)
    m, win, dt = 64, 32, 0.1
    reach = F((m + win + 8) * dt + 1e-6)
    qa = moved_axis(ql, qd, qw, s0.astype(F))
    qz = moved_axis(ql, qd, qw, (s0 + ln - 1).astype(F))
    sl = wslack(np.fmin(qa[0], qz[0]), np.fmax(qa[1], qz[1]), reach)
    sl = F(slack) * (sl + F(along) * (np.abs(a) * sl[rows, k]).astype(F)).astype(F)
    qa, qz = _shear(*qa, a, k), _shear(*qz, a, k)
    da, dz = (s0 - r).astype(F), (s0 + ln - 1 - r).astype(F)
    wl = np.fmin(((qa[0] - np.fmax(da * glo, da * ghi)).astype(F) - sl).astype(F),
                 ((qz[0] - np.fmax(dz * glo, dz * ghi)).astype(F) - sl).astype(F))
    wh = np.fmax(((qa[1] - np.fmin(da * glo, da * ghi)).astype(F) + sl).astype(F),
                 ((qz[1] - np.fmin(dz * glo, dz * ghi)).astype(F) + sl).astype(F))
    tr = _shear(*moved_axis(tl, td, tw, r.astype(F)), a, k)
    met = exact_hits(q, t, s0, ln).any(axis=1)
    return met, met & ~((tr[0] <= wh) & (tr[1] >= wl)).all(axis=1)


def test_hull_holds_leaves_that_just_touch():
    met, out = _outside(1.0)
    assert met.sum() > 20_000
    assert not out.any(), f"{out.sum()} leaves met outside the sheared hull"


def test_half_is_to_spare():
    assert not _outside(0.5)[1].any()


def test_no_slack_loses_leaves():
    assert _outside(0.0)[1].any()


def test_slack_of_the_own_axis_alone_loses_leaves():
    assert _outside(1.0, along=0.0)[1].any()
