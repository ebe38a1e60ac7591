"""Counters of a pass with coincident particles: their pairs are left out of
every count, so that the sign tests are those of the pairs counted (one for a
pair before the history, else one and the halvings of D - 1 slots)."""
import math

import pytest

from paper_2605_05543_amd import _lib, bunch

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("depth", [2, 3, 100, 257])
def test_coincident_pairs_are_not_counted(depth, precision):
    print(f"case counters depth={depth} precision={precision}", flush=True)
    n = 70
    r, u = bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), 1.0, seed=3))
    r[:, 5], u[:, 5] = r[:, 2], u[:, 2]
    with _lib.Context(n=n, depth=depth, q=Q, m=ME, dt=51.2e-12 / depth, precision=precision) as ctx:
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()
        ctx.set_counting(True)
        ctx.step(1)
        c = ctx.counters()
        with pytest.raises(_lib.EmppError):
            ctx.sync()
    assert c["pairs"] == n * (n - 1) - 2
    halvings = math.ceil(math.log2(depth - 1)) if depth > 2 else 0
    assert c["probes"] == c["before"] + (c["pairs"] - c["before"]) * (1 + halvings)
