"""Cooperative launches whose waits give up (a limit of no polls, set on the
context): the call reports EDEVICE, what it leaves is not taken for valid by later
calls, and after a fresh start the context gives what another one gives."""
import ctypes

import numpy as np
import pytest

from paper_2605_05543_amd import _lib, bunch

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON


def _wait_polls(ctx, polls):
    _lib.lib.empp_internal_wait_polls(ctx.h, ctypes.c_uint32(polls))


@pytest.mark.parametrize("steps", [30, 5000])
def test_transport_that_gives_up(steps):
    print(f"case transport gives up steps={steps}", flush=True)
    n = 20000
    rng = np.random.default_rng(4)
    r = 1e-3 * rng.standard_normal((3, n))
    r[0] += 3 * bunch.R_EARTH
    u = 3e8 * (0.1 * rng.standard_normal((3, n)) + np.array([[0.0], [1.0], [1.5]]))
    kw = dict(n=n, depth=2, q=Q, m=ME, dt=1e-13, ext_field=1, dipole_b0=3.12e-5, dipole_re=bunch.R_EARTH)

    def run(ctx):
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()
        ctx.handoff()
        ctx.transport(1e-7, 1 / 32, 20)
        return ctx.state()

    with _lib.Context(**kw) as ctx:
        ref = run(ctx)
    with _lib.Context(**kw) as ctx:
        run(ctx)
        _wait_polls(ctx, 0)
        with pytest.raises(_lib.EmppError) as ei:
            ctx.transport(1e-7, 1 / 32, steps)
        assert ei.value.status == _lib.EMPP_EDEVICE
        _wait_polls(ctx, 1 << 24)
        for call in (lambda: ctx.transport(1e-7, 1 / 32, 6), ctx.state, ctx.diag, ctx.handoff):
            with pytest.raises(_lib.EmppError) as ei:
                call()
            assert ei.value.status == _lib.EMPP_ESTATE
        for a, b in zip(ref, run(ctx)):
            assert np.array_equal(a, b)
