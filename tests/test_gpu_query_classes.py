"""Queries ordered by energy class within their cells (broad spectra, one instance): the candidates,
hits and pairs must be those of one launch per step, whose queries are in plain Morton order, also
where the rule falls just short (narrow or weak beams) and where almost every query is below
threshold."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1608_01125_amd import beams

from test_gpu_window import _run, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("par", [(0.1, 10.0), (0.01, 3.9), (0.01, 4.3), (0.002, 0.6), (30.0, 300.0)])
def test_order_by_class_keeps_candidates(torch, par):  # noqa: F811
    """(0.01, 3.9) and (0.01, 4.3) MeV: E_max^2 / m_e^2 = 58 and 71, on the two sides of 64."""
    wl = beams.broadband_16m(n=6000, w=3e14)
    wl = replace(wl, a=replace(wl.a, e_par=par), b=replace(wl.b, e_par=par))
    A, B = beams.draw_pair(wl)
    base, cand1 = _run(wl, A, B, 400, 150, 1, 1)
    got, cand = _run(wl, A, B, 400, 150, 40, 0)
    assert got[3]["n_candidates"] == base[3]["n_candidates"]
    for f in ("n_hits", "n_pairs"):
        assert got[3][f] == base[3][f]
    for a, b in zip(got[:3], base[:3]):
        assert np.array_equal(a, b)
    if par[1] > 1.0:
        assert base[3]["n_candidates"] > 0
