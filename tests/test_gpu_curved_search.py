"""The search of a wavefront whose guesses miss, on strongly curved histories:
depths on both sides of every batch of halvings and with one, two and many tiles,
spans that leave none, some and most pairs before the history, target counts that
leave lanes without a target.  k* against the oracle, exactly, from the plain
bisection and from a guess; the fields of every mode and path bit for bit with
those of the plain bisection's brackets, so that every bracket is the same.  (Fields
against the oracle are other tests': a segment of 25 ps of these paths is so
coarse that rounding alone exceeds the tolerance.)"""
import numpy as np
import pytest

import oracle
from paper_2605_05543_amd import bunch
from parity import assert_kstar
from test_gpu_lone_target import gyrating_history

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("depth", [2, 3, 4, 5, 6, 9, 10, 17, 18, 33, 34, 130, 300, 2047, 2049])
@pytest.mark.parametrize("span", [51.2e-12, 8e-12])
def test_searches_agree(precision, depth, span):
    from paper_2605_05543_amd._lib import Context

    print(f"case curved search depth={depth} span={span} precision={precision}", flush=True)
    n, m = 150, 129
    T, w, v, u = gyrating_history(n, depth, span, 1.5, seed=depth)
    rng = np.random.default_rng(depth)
    x = 1.2e-3 * rng.standard_normal((3, m))
    si = np.full(m, -1)
    x[:, -1], si[-1] = w[-1][:, 70], 70  # alone in its wavefront, and a source
    x[:, 5], si[5] = w[-1][:, 3], 3
    orc = oracle.get()
    k0 = orc.fields(T, w, v, Q, T[-1], x, si, want_kstar=True)[2]
    for splits in (1, 0):
        with Context(n=n, depth=depth, q=Q, m=ME, dt=span / depth, source_splits=splits) as ctx:
            ctx.set_history(T, w, v, u)
            out = []
            for guess in (0, 2):
                ctx.set_mode(precision, guess)
                E, B = ctx.fields_at(T[-1], x, si)
                E1, B1, k = ctx.fields_at(T[-1], x, si, want_kstar=True)
                assert_kstar(f"guess={guess}", k, k0)
                out += [(E, B), (E1, B1)]
            assert all(np.array_equal(a, b) for o in out for a, b in zip(out[0], o))
