"""Swarms without relative motion: photons of one direction whose |p| falls short of E by half the
1e-12 that photon data may, energetic enough to be above threshold. What lies within r at the
window's start collides, counts as the brute-force oracle's."""
import numpy as np
import pytest

from test_gpu_swarm import _check, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _parallel(seed, n, E, d):
    rng = np.random.default_rng(seed)
    b = {f: rng.normal(0.0, 1.5e-9, n) for f in ("x", "y", "z")}
    b["E"] = np.asarray(E) * np.ones(n)
    for a, f in enumerate(("px", "py", "pz")):
        b[f] = b["E"] * (d[a] * (1.0 - 5e-13))
    b["w"] = rng.integers(30, 700, n).astype(float)
    return b


@pytest.mark.parametrize("d", [(0.0, 0.0, 1.0), (0.6, 0.0, 0.8), (0.0, -1.0, 0.0)])
@pytest.mark.parametrize("energies", [2e6, [1e6, 1.7e6, 2e6, 3.1e6, 4.7e6]])
def test_photons_of_one_direction(torch, energies, d):  # noqa: F811
    A, B = _parallel(1, 5, energies, d), _parallel(2, 5, energies, d)
    for k0 in (0, 3):
        cnt = _check(torch, A, B, (4e-9, 4e-9, 4e-9), k0=k0)
        assert (cnt > 0).sum() > 10
