"""Swarms by blocks of 64 real photons against the brute-force oracle, counts identical: swarms
of several octree levels (nodes dropped, counted whole and descended), counts about a block and
a level, windows that end within the crossing (every approach of a pair cut off), and swarms
that meet far from the origin, where more pairs lie within the positions' rounding of r."""
import numpy as np
import pytest

from test_gpu_swarm import _check, _tiny, torch  # noqa: F401

pytestmark = pytest.mark.gpu
CELL = (4e-9, 4e-9, 4e-9)


@pytest.mark.parametrize("wa,wb,cell", [
    ([63.0, 64.0, 65.0], [4097.0, 20000.0, 1.0], CELL),
    ([20000.0, 512.0, 513.0], [20000.0, 7.0, 511.0], CELL),
    ([5000.0, 300.0, 1.0], [3000.0, 64.0, 8.0], (2e-8, 3e-9, 9e-9))])
def test_sizes_and_levels(torch, wa, wb, cell):  # noqa: F811
    A, B = _tiny(21, 3, spread=1e-9, along=1e-3)
    A["w"], B["w"] = np.array(wa), np.array(wb)
    _check(torch, A, B, cell)


@pytest.mark.parametrize("phi,along", [(180.0, 1.5e-9), (90.0, 1.5e-9), (180.0, 0.0)])
@pytest.mark.parametrize("k0,n_steps", [(0, 5), (5, 3)])
def test_window_ends_within_the_crossing(torch, phi, along, k0, n_steps):  # noqa: F811
    """The clouds' centres meet at t = 0.5, the end (or the start) of the window."""
    A, B = _tiny(22, 5, phi_deg=phi, along=along, spread=1.5e-9, w_lo=100, w_hi=700)
    _check(torch, A, B, CELL, k0=k0, n_steps=n_steps, min_total=0)


def test_far_from_the_origin(torch):  # noqa: F811
    A, B = _tiny(23, 6, along=0.02, w_lo=200, w_hi=700)
    for b in (A, B):
        b["x"] += 30.0
        b["y"] -= 50.0
    _check(torch, A, B, CELL)
