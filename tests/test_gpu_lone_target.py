"""A wavefront with one target, whose own source comes while the wavefront
bisects without a guess (histories that curve so that guesses miss in a row):
the pair is left out and no bracket of it is needed, with and without the slot
table (D up to 2048 and beyond), in both precisions and in a step.  Against the
oracle; tolerances those of every field (parity.FP64_TOL, parity.MIXED_TOL)."""
import numpy as np
import pytest

import oracle
from paper_2605_05543_amd import bunch
from parity import assert_fields, assert_mixed

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON


def gyrating_history(n, depth, span, turn, seed):
    """A 1 MeV bunch turning by `turn` rad over the stored history."""
    r, u = bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), 1.0, seed=seed))
    u = bunch.beam_rotation(np.pi / 2, np.pi / 2) @ u
    vel = u / np.sqrt(1.0 + (u * u).sum(0) / bunch.C_LIGHT**2)
    T = span / depth * np.arange(-(depth - 1), 1, dtype=np.float64)
    ca, sa = np.cos(turn * T / span), np.sin(turn * T / span)
    v = np.stack([ca[:, None] * vel[0] - sa[:, None] * vel[1], sa[:, None] * vel[0] + ca[:, None] * vel[1],
                  np.broadcast_to(vel[2], (depth, n))], axis=1)
    w = np.empty((depth, 3, n))
    w[-1] = r
    for k in range(depth - 2, -1, -1):
        w[k] = w[k + 1] - v[k] * (T[k + 1] - T[k])
    v[-1] = v[-2]
    gam = np.sqrt(1.0 + (u * u).sum(0) / bunch.C_LIGHT**2)
    return T, w, v, gam * v[-1]


@pytest.mark.parametrize("depth", [1500, 3000])
@pytest.mark.parametrize("precision", [0, 1])
def test_own_source_among_misses(depth, precision):
    from paper_2605_05543_amd._lib import Context

    print(f"case lone target depth={depth} precision={precision}", flush=True)
    n = 65
    T, w, v, u = gyrating_history(n, depth, 51.2e-12, 1.5, seed=depth)
    check = assert_mixed if precision else assert_fields
    orc = oracle.get()
    E0, B0, SE, SB = orc.fields(T, w, v, Q, T[-1], w[-1], np.arange(n), want_abs=True)
    with Context(n=n, depth=depth, q=Q, m=ME, dt=51.2e-12 / depth, precision=precision, source_splits=1) as ctx:
        ctx.set_history(T, w, v, u)
        got = [ctx.fields_at(T[-1], w[-1][:, i:i + 1], np.array([i])) for i in range(n)]
        E, B = (np.concatenate([g[k] for g in got], axis=1) for k in (0, 1))
        check("one target a call", E, B, E0, B0, SE, SB)
        ctx.step(1)
        check("step", *ctx.fields(), E0, B0, SE, SB)
