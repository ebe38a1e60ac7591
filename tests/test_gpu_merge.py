"""The merge of the source chunks' partials (16 wavefronts per 64 targets up
to 16384 targets, four beyond) against the oracle: field calls and steps at
the edges of its 64-target blocks, with fewer, as many and more chunks than
wavefronts.  Tolerance: that of every FP64 field (parity.FP64_TOL)."""
import numpy as np
import pytest

import oracle
from paper_2605_05543_amd import bunch
from parity import assert_fields

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON


@pytest.mark.parametrize("n,splits", [(63, 1), (64, 16), (65, 17), (130, 33), (16384, 3), (16385, 0)])
def test_merge_of_chunks(n, splits):
    from paper_2605_05543_amd._lib import Context

    print(f"case merge n={n} chunks={splits}", flush=True)
    depth, dt = 8, 1e-12
    orc = oracle.get()
    r, u = bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), 1.0, seed=n))
    sub = bunch.target_subset(n, 64, 9)
    sub[-1] = n - 1
    T, w, v = orc.init_straight(r, u, depth, dt)
    E0, B0, SE, SB = orc.fields(T, w, v, Q, T[-1], r[:, sub], sub, want_abs=True)
    with Context(n=n, depth=depth, q=Q, m=ME, dt=dt, source_splits=splits) as ctx:
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()
        Ef, Bf = ctx.fields_at(0.0, r, np.arange(n))
        ctx.step(1)
        Es, Bs = ctx.fields()
    assert_fields("fields_at", Ef[:, sub], Bf[:, sub], E0, B0, SE, SB)
    assert_fields("step", Es[:, sub], Bs[:, sub], E0, B0, SE, SB)
