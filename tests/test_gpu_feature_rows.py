"""Feature rows in buffers of the caller's size: a call whose rows do not fit reports their number
and keeps the pairs, tril_st_feature_rows then forms the same rows; the binding's tensors hold
them exactly, whatever capacity it was given."""
import ctypes

import pytest

from paper_1608_01125_amd import beams, surrogate
from paper_1608_01125_amd import tril as T

from test_gpu_st_window import torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def instance(torch):  # noqa: F811
    inst = surrogate.Instance(beams.st_train_instance(4, 600))
    ctx = T.Context(inst.wl.dt, None)
    yield inst, ctx, inst.features(ctx)
    ctx.close()


def _room(torch, n):  # noqa: F811
    return (torch.zeros((n, 6), dtype=torch.float32, device="cuda"),
            torch.zeros(n, dtype=torch.float64, device="cuda"),
            torch.zeros(n, dtype=torch.int64, device="cuda"))


def _features(inst, ctx, out, cap, steps=None):
    n = ctypes.c_int64(-1)
    gq, gt, p = T.st_grid(inst.ga), T.st_grid(inst.gb), T.sur_params()
    code = T.lib().tril_st_features(
        ctx.h, inst.qsums.data_ptr(), ctypes.byref(gq), inst.tsums.data_ptr(), ctypes.byref(gt), 0,
        inst.wl.n_steps if steps is None else steps, ctypes.byref(p),
        *(v.data_ptr() if cap else None for v in out), cap, ctypes.byref(n))
    return code, n.value


def _rows(inst, ctx, out, n, swap=False):
    gq, gt = T.st_grid(inst.ga), T.st_grid(inst.gb)
    if swap:
        gq.n_e = 2
    return T.lib().tril_st_feature_rows(ctx.h, inst.qsums.data_ptr(), ctypes.byref(gq),
                                        inst.tsums.data_ptr(), ctypes.byref(gt),
                                        *(v.data_ptr() for v in out), n)


def _same(torch, got, want):  # noqa: F811
    """Keys equal; y0 and the features within what the order of the additions to a pair's overlap
    may do: below 1000 positive terms, 1000 x 2^-53 relative, and one rounding of the FP32 log."""
    assert torch.equal(got[2], want[2])
    torch.testing.assert_close(got[1], want[1], rtol=1.2e-13, atol=0.0)
    torch.testing.assert_close(got[0], want[0], rtol=2.0 ** -23, atol=1.2e-13)


def test_binding_returns_the_rows_alone(torch, instance):  # noqa: F811
    inst, ctx, want = instance
    n = want[2].shape[0]
    assert n > 1000
    for cap in (0, 1, n - 1, n, 1 << 20):
        got = T.tril_st_features(ctx, inst.qsums, inst.ga, inst.tsums, inst.gb, 0,
                                 inst.wl.n_steps, None, cap)
        _same(torch, got, want)
        assert [v.untyped_storage().nbytes() for v in got] == [24 * n, 8 * n, 8 * n]
    empty = T.tril_st_features(ctx, inst.qsums, inst.ga, inst.tsums, inst.gb, 0, 0)
    assert [tuple(v.shape) for v in empty] == [(0, 6), (0,), (0,)]
    with pytest.raises(T.TrilError) as ei:
        T.tril_st_features(ctx, inst.qsums, inst.ga, inst.tsums, inst.gb, 0, 1, None, -1)
    assert ei.value.code == T.TRIL_E_INVAL


@pytest.mark.parametrize("short", [0, 1, 1000])
def test_rows_after_an_overflow(torch, instance, short):  # noqa: F811
    inst, ctx, want = instance
    n = want[2].shape[0]
    cap = n - short if short else n
    out = _room(torch, n)
    code, rows = _features(inst, ctx, out, cap)
    assert rows == n
    if short == 0:
        assert code == T.TRIL_OK and _rows(inst, ctx, out, n) == T.TRIL_E_STATE
    else:
        assert code == T.TRIL_E_OVERFLOW
        assert _rows(inst, ctx, out, n - 1) == T.TRIL_E_STATE
        assert _rows(inst, ctx, out, n, swap=True) == T.TRIL_E_STATE
        assert _rows(inst, ctx, out, n) == T.TRIL_OK
        assert _rows(inst, ctx, out, n) == T.TRIL_E_STATE  # given once
    _same(torch, out, want)


def test_pairs_are_those_of_the_last_call(torch, instance):  # noqa: F811
    """A later call that forms features ends the wait, its own overflow begins another."""
    inst, ctx, want = instance
    n = want[2].shape[0]
    out = _room(torch, n)
    assert _features(inst, ctx, out, 0) == (T.TRIL_E_OVERFLOW, n)
    inst.audit(ctx, None, T.AUDIT_BIN_LEVEL, 200, 2, 1)
    assert _rows(inst, ctx, out, n) == T.TRIL_E_STATE
    code, part = _features(inst, ctx, out, 0, inst.wl.n_steps // 2)
    assert code == T.TRIL_E_OVERFLOW and 0 < part < n
    assert _rows(inst, ctx, out, n) == T.TRIL_E_STATE
    assert _rows(inst, ctx, out, part) == T.TRIL_OK
    assert torch.equal(out[2][part:], torch.zeros(n - part, dtype=torch.int64, device="cuda"))
    assert (out[2][1:part] > out[2][:part - 1]).all()
