"""The hull of a descent over sheared node boxes (host check, no GPU).

Node boxes are formed in the coordinates x_i - a_i x_k (|a_i| <= 1, a_k = 0): the box of a leaf
at the copy's step r, and the query's boxes at the descent's first and last steps, are taken to
the intervals of their points in those coordinates, and the query's are widened by the sheared
motion bounds and by the slack of axis i plus |a_i| that of axis k. Any leaf whose box at a step
of the descent meets the query's box there must have its sheared box at r inside the hull. The
device's FP32 steps are emulated; the forms without the slack and with the shear of the motion
left out must fail somewhere, so that the check has teeth."""
import numpy as np

from test_descent_bounds import F, _pairs, exact_hits, moved_axis, wslack


def _shear(lo, hi, a, k):
    rows = np.arange(lo.shape[0])[:, None]
    e = (a * lo[rows, k]).astype(F)
    f = (a * hi[rows, k]).astype(F)
    return (lo - np.fmax(e, f)).astype(F), (hi - np.fmin(e, f)).astype(F)


def _misses(slack=1.0, motion=True, n=60_000, seed=37):
    rng = np.random.default_rng(seed)
    q, t, s0, ln = _pairs(n, seed)
    (ql, qd, qw), (tl, td, tw) = q, t
    k = rng.integers(0, 3, size=(n, 1))
    rows = np.arange(n)[:, None]
    a = rng.uniform(-1, 1, size=(n, 3)) * 10.0 ** rng.choice([0, 0, -3, -7], size=(n, 1))
    a[rng.random((n, 3)) < 0.2] = 1.0
    a = a.astype(F)
    a[rows, k] = 0.0
    spread = np.where(rng.random((n, 1)) < 0.5, 0.0, rng.uniform(0, 0.5, size=(n, 1))).astype(F)
    vlo = np.nextafter((td - np.abs(td) * spread).astype(F), F(-np.inf))
    vhi = np.nextafter((td + np.abs(td) * spread).astype(F), F(np.inf))
    if motion:  # the sheared motion's bounds, formed in FP64 and rounded outward
        e = a.astype(np.float64) * vlo[rows, k]
        f = a.astype(np.float64) * vhi[rows, k]
        on = a != 0
        glo = np.where(on, np.nextafter((vlo - np.fmax(e, f)).astype(F), F(-np.inf)), vlo)
        ghi = np.where(on, np.nextafter((vhi - np.fmin(e, f)).astype(F), F(np.inf)), vhi)
    else:
        glo, ghi = vlo, vhi
    r = s0 + rng.integers(-16, 48, size=(n, 1)) % np.maximum(ln + 16, 1)
    m, win, dt = 4096 + 32, 32, 0.1  # every motion per step is at most 0.1
    reach = F((m + win + 8) * dt + 1e-6)
    qa = moved_axis(ql, qd, qw, s0.astype(F))
    qz = moved_axis(ql, qd, qw, (s0 + ln - 1).astype(F))
    sl = wslack(np.fmin(qa[0], qz[0]), np.fmax(qa[1], qz[1]), reach)
    sl = F(slack) * (sl + (np.abs(a) * sl[rows, k]).astype(F)).astype(F)
    qa, qz = _shear(*qa, a, k), _shear(*qz, a, k)
    da, dz = (s0 - r).astype(F), (s0 + ln - 1 - r).astype(F)
    wl = np.fmin(((qa[0] - np.fmax(da * glo, da * ghi)).astype(F) - sl).astype(F),
                 ((qz[0] - np.fmax(dz * glo, dz * ghi)).astype(F) - sl).astype(F))
    wh = np.fmax(((qa[1] - np.fmin(da * glo, da * ghi)).astype(F) + sl).astype(F),
                 ((qz[1] - np.fmin(dz * glo, dz * ghi)).astype(F) + sl).astype(F))
    tr = _shear(*moved_axis(tl, td, tw, r.astype(F)), a, k)
    met = exact_hits(q, t, s0, ln).any(axis=1)
    inside = ((tr[0] <= wh) & (tr[1] >= wl)).all(axis=1)
    return met, met & ~inside


def test_sheared_hull_holds_every_leaf_met():
    met, miss = _misses()
    assert met.sum() > 10_000
    assert not miss.any(), f"{miss.sum()} leaves met outside the sheared hull"


def test_half_the_slack_suffices():
    assert not _misses(slack=0.5)[1].any()


def test_unsheared_motion_loses_leaves():
    assert _misses(motion=False)[1].any()
