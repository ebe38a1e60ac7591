"""Indices of a device field call: a self_index that names no source leaves none
out, whatever its low bits, and an error names the target's index in the call."""
import numpy as np
import pytest

from paper_2605_05543_amd import _lib, bunch
from test_zz_no_alloc import _fields

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON
CALLS = (_lib.empp_fields_at_dev, _lib.empp_fields_at_dev_noalloc)


def _context(n, depth, precision):
    T, w, v = bunch.wiggly_history(n, depth, 1e-13, beta=0.9, accel_rel=0.1, seed=5)
    ctx = _lib.Context(n=n, depth=depth, q=Q, m=ME, dt=1e-13, precision=precision)
    ctx.set_history(T, w, v, np.zeros((3, n)))
    return ctx, T, w


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("fn", CALLS)
def test_self_index_beyond_the_sources(fn, precision):
    print(f"case self_index beyond the sources precision={precision}", flush=True)
    ctx, T, w = _context(40, 16, precision)
    with ctx:
        x = 1.5e-3 * np.random.default_rng(1).standard_normal((3, 70))
        ref = _fields(fn, ctx, T[-1], x, np.full(70, -1))
        for base in (1 << 32, -(1 << 32), 1 << 40, 40):
            got = _fields(fn, ctx, T[-1], x, base + np.arange(70) % 40)
            assert all(np.array_equal(a, b) for a, b in zip(ref, got)), base


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("fn", CALLS)
def test_errors_name_the_calls_target(fn, precision):
    print(f"case error in a later part of a call precision={precision}", flush=True)
    n = 40
    ctx, T, w = _context(n, 16, precision)
    with ctx:
        for at in ((3,), (n + 5,), (2 * n + 1, 3 * n - 1)):
            x = 1.5e-3 * np.random.default_rng(1).standard_normal((3, 3 * n))
            x[:, at] = w[-1][:, 7:8]  # on a source that is not left out
            with pytest.raises(_lib.EmppError, match=f"target {at[0]}, source 7") as ei:
                _fields(fn, ctx, T[-1], x, np.full(3 * n, -1))
            assert ei.value.status == _lib.EMPP_ENUMERIC
