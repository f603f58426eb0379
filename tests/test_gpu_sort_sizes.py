"""The radix sort at the sizes where its route changes (one workgroup up to 8192 keys, tiles of
1024 up to 245760, tiles of 4096 above) and at its tiles' ends, for both key widths and every
number of passes, against numpy's stable order."""
import numpy as np
import pytest

from test_gpu_kernels import _sort_case, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 8191, 8192, 8193,
                               9216, 245759, 245760, 245761, 262144, 262145])
def test_sizes_about_the_routes(torch, n, wide):  # noqa: F811
    rng = np.random.default_rng(n)
    keys = rng.integers(0, 1 << 20, n, dtype=np.uint64)  # many ties: the order has to be stable
    _sort_case(torch, keys if wide else keys.astype(np.uint32), 20, wide)


@pytest.mark.parametrize("bits", [1, 8, 9, 24, 32, 40, 64])
@pytest.mark.parametrize("n", [777, 5000, 20000])
def test_passes(torch, n, bits):  # noqa: F811
    rng = np.random.default_rng(bits)
    keys = rng.integers(0, 1 << 63, n, dtype=np.uint64) * np.uint64(2) + np.uint64(1)
    keys = keys & np.uint64((1 << bits) - 1)
    _sort_case(torch, keys, bits, True)
    if bits <= 32:
        _sort_case(torch, keys.astype(np.uint32), bits, False)
