"""Clouds that move a cell and more per step: windows shorter than 32 steps, down to one whose
boxes are those of the mid-step alone; every bin-pair yield against the oracle."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1608_01125_amd import beams

from test_gpu_st_window import _check, _reference, _table, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("phi", [180.0, 90.0, 40.0])
@pytest.mark.parametrize("factor,step_batch", [(2, 0), (5, 0), (5, 4), (11, 0), (32, 0), (33, 0),
                                               (200, 0)])
def test_fast_clouds(torch, factor, phi, step_batch):  # noqa: F811
    wl = beams.st_headon(1500, seed=8)
    wl = replace(wl, b=replace(wl.b, phi_deg=phi), dt=wl.dt * factor, n_steps=wl.n_steps // factor)
    A, B = beams.draw_pair(wl)
    ga, gb = beams.st_grid(wl, "a", A), beams.st_grid(wl, "b", B)
    assert min(ga.cell) == pytest.approx(0.5)
    k0, n_steps = wl.n_steps // 3, wl.n_steps - wl.n_steps // 3
    got = _table(torch, A, B, ga, gb, wl, k0, n_steps, step_batch=step_batch)
    ref = _reference(A, B, ga, gb, wl, k0, n_steps, [0, 1500], [0, 1500])
    assert ref[1] > 0
    _check(got, ref)
