"""Host field calls after a step that failed: the step's error comes before any
other, the outputs stay as they were, whatever block they would have come through,
and with counting on the refused call's pairs are not counted."""
import numpy as np
import pytest

from paper_2605_05543_amd import _lib, bunch

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON


@pytest.mark.parametrize("m,kstar,index,counting", [
    (4, True, None, False), (4, False, "bad", False), (4, True, None, True),
    (200000, True, None, False), (30000, True, "good", False), (200000, False, "bad", False),
])
def test_the_earlier_error_comes_first(m, kstar, index, counting):
    print(f"case earlier error first m={m} kstar={kstar} index={index} counting={counting}", flush=True)
    n = 64
    r, u = bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), 1.0, seed=3))
    r[:, 5], u[:, 5] = r[:, 2], u[:, 2]  # coincident particles
    x = np.ascontiguousarray(r[:, :1] + 1e-3 * (1.0 + np.arange(m) / m))
    si = None if index is None else np.full(m, -1 if index == "good" else n)
    E, B, k = np.full((3, m), 7.0), np.full((3, m), 7.0), np.full((m, n), 7, np.int32)

    def call(si):
        return _lib.lib.empp_fields_at(ctx.h, 1e-13, m, _lib._ptr(x), _lib._ptr(si), _lib._ptr(E), _lib._ptr(B),
                                       _lib._ptr(k) if kstar else None)

    with _lib.Context(n=n, depth=4, q=Q, m=ME, dt=1e-13) as ctx:
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()
        ctx.step(1)
        ctx.set_counting(counting)
        assert call(si) == _lib.EMPP_ENUMERIC
        assert b"an earlier step: coincident particles" in _lib.lib.empp_last_error()
        assert np.all(E == 7.0) and np.all(B == 7.0) and np.all(k == 7)
        assert ctx.counters()["pairs"] == 0
        if index == "bad":
            assert call(si) == _lib.EMPP_EINVAL
        assert call(None) == _lib.EMPP_OK  # the error is reported once
        assert np.all(E != 7.0) and (not kstar or np.all(k != 7))
        assert ctx.counters()["pairs"] == (m * n if counting else 0)
