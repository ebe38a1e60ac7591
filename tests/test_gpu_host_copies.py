"""Read-backs and host field calls through the context's kept blocks and
beyond them: host calls bit-identical to device calls on the same context
while the blocks grow, shrink and are passed by (outputs alone or k* too
large), state and fields of small and large bunches, and an error of an
earlier step reported as such."""
import numpy as np
import pytest

import oracle
from paper_2605_05543_amd import bunch
from parity import assert_fields
from test_zz_no_alloc import _fields

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON


def test_host_field_calls():
    from paper_2605_05543_amd import _lib

    print("case host field calls", flush=True)
    n, depth, dt = 65, 8, 1e-13
    T, w, v = bunch.wiggly_history(n, depth, dt, beta=0.9, accel_rel=0.1, seed=1)
    rng = np.random.default_rng(2)
    with _lib.Context(n=n, depth=depth, q=Q, m=ME, dt=dt) as ctx:
        ctx.set_history(T, w, v, np.zeros((3, n)))
        for m in (5, 3001, 1, 20000, 7, 60000, 70000, 301):
            x = 1.5e-3 * rng.standard_normal((3, m))
            si = np.full(m, -1, np.int64)
            x[:, 0], si[0] = w[-1][:, 3], 3
            E, B, k = _fields(_lib.empp_fields_at_dev, ctx, T[-1], x, si)
            E1, B1, k1 = ctx.fields_at(T[-1], x, si, want_kstar=True)
            E2, B2 = ctx.fields_at(T[-1], x, si)
            assert np.array_equal(E, E1) and np.array_equal(B, B1) and np.array_equal(k, k1), m
            assert np.array_equal(E, E2) and np.array_equal(B, B2), m
        E3, B3 = ctx.fields_at(T[-1], x + 1e-3)
        assert E3.shape == x.shape and np.all(np.isfinite(E3)) and np.all(np.isfinite(B3))


@pytest.mark.parametrize("n", [2, 33, 100000])
def test_state_and_fields(n):
    from paper_2605_05543_amd._lib import Context

    print(f"case read-back n={n}", flush=True)
    depth, dt = 2, 1e-13
    orc = oracle.get()
    r, u = bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), 1.0, seed=n))
    sub = np.unique(np.r_[0, n - 1, np.arange(0, n, max(1, n // 16))])
    T, w, v = orc.init_straight(r, u, depth, dt)
    E0, B0, SE, SB = orc.fields(T, w, v, Q, T[-1], r[:, sub], sub, want_abs=True)
    with Context(n=n, depth=depth, q=Q, m=ME, dt=dt) as ctx:
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()
        rg, ug, t, step = ctx.state()
        assert np.array_equal(rg, r) and np.array_equal(ug, u) and (t, step) == (0.0, 0)
        ctx.step(1)
        E, B = ctx.fields()
        assert ctx.state()[3] == 1
    assert_fields("step", E[:, sub], B[:, sub], E0, B0, SE, SB)


@pytest.mark.parametrize("m", [4, 70000])
def test_an_earlier_steps_error(m):
    from paper_2605_05543_amd import _lib

    print(f"case earlier error m={m}", flush=True)
    n = 8
    r, u = bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), 1.0, seed=3))
    r[:, 5], u[:, 5] = r[:, 2], u[:, 2]  # coincident particles
    x = r[:, :1] + 1e-3 * np.arange(1, m + 1)
    with _lib.Context(n=n, depth=4, q=Q, m=ME, dt=1e-13) as ctx:
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()
        E, _ = ctx.fields_at(0.0, x)  # external targets see no coincidence
        assert np.all(np.isfinite(E))
        ctx.step(1)
        with pytest.raises(_lib.EmppError, match="an earlier step") as ei:
            ctx.fields_at(1e-13, x)
        assert ei.value.status == _lib.EMPP_ENUMERIC
        for call in (ctx.fields, ctx.state):
            call()  # reported once
            ctx.step(1)
            with pytest.raises(_lib.EmppError):
                call()
