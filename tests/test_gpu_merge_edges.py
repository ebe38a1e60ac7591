"""The merge of the source chunks' partials at the edges of its blocks: 15, 16 and
17 targets for those of 16 (up to 16384 targets), 7, 8 and 9 chunks for a step's
eight slices, 31, 32 and 33 for a field call's.  Against one chunk, whose fields
other tests hold against the oracle: the pairs' fields are the same bits, so the
sums differ by their additions' rounding alone, at most twice the 31 of a plain
partial and four compensated ones, 70 u = 7.8e-15 of the sum of magnitudes a
component, 1.4e-14 as a vector.  Bound 2e-14."""
import numpy as np
import pytest

import oracle
from paper_2605_05543_amd import bunch

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON
TOL = 2e-14


def _run(r, u, depth, dt, splits, ms):
    from paper_2605_05543_amd._lib import Context

    n = r.shape[1]
    with Context(n=n, depth=depth, q=Q, m=ME, dt=dt, source_splits=splits) as ctx:
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()
        out = [ctx.fields_at(0.0, r[:, :m], np.arange(m)) for m in ms]
        ctx.step(1)
        return out + [ctx.fields()]


@pytest.mark.parametrize("n,splits", [(113, 7), (128, 8), (145, 9), (497, 31), (512, 32), (529, 33), (15, 9), (16, 9),
                                      (17, 9), (17, 0)])
def test_merge_at_its_edges(n, splits):
    print(f"case merge edges n={n} chunks={splits}", flush=True)
    depth, dt = 8, 1e-12
    orc = oracle.get()
    r, u = bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), 1.0, seed=n))
    T, w, v = orc.init_straight(r, u, depth, dt)
    _, _, SE, SB = orc.fields(T, w, v, Q, T[-1], r, np.arange(n), want_abs=True)
    ms = [m for m in (15, 16, 17, n) if m <= n]
    for (E, B), (E1, B1) in zip(_run(r, u, depth, dt, splits, ms), _run(r, u, depth, dt, 1, ms)):
        m = E.shape[1]
        e, b = (np.max(np.linalg.norm(x - y, axis=0) / S[:m]) for x, y, S in ((E, E1, SE), (B, B1, SB)))
        print(f"   m={m}: {e:.1e} {b:.1e} of the sum of magnitudes", flush=True)
        assert e <= TOL and b <= TOL
