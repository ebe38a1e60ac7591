"""The cut of a pair launch (wavefronts that share a target's sources, source
chunks) against the oracle: target counts at the edges of 1 ... 16 wavefronts
of targets and beyond the particle count, tiles of 16, 4, 2 and 1 sources,
fewer sources than wavefronts, and histories that the chord guess meets and
misses for many sources in a row.  Fields with and without k*, of the
allocation-free call and of every search mode that shares the launch are
bit-identical.  Tolerances: those of every field (parity.FP64_TOL,
parity.MIXED_TOL)."""
import numpy as np
import pytest

import oracle
from paper_2605_05543_amd import bunch
from parity import assert_fields, assert_kstar, assert_mixed
from test_zz_no_alloc import _fields

pytestmark = pytest.mark.gpu

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON


@pytest.mark.parametrize("precision,n,depth,accel,ms", [
    (0, 3, 8, 0.1, (1, 7)),
    (0, 90, 128, 0.1, (1, 64, 65, 200)),
    (0, 700, 512, 0.0, (63, 129, 257, 700, 1500)),
    (0, 700, 600, 0.3, (64, 300, 513)),
    (0, 130, 1100, 0.1, (64, 130)),
    (0, 70, 2048, 0.1, (1, 130)),
    (1, 90, 128, 0.1, (1, 200)),
    (1, 700, 512, 0.0, (64, 700, 1500)),
])
def test_split_of_a_launch(precision, n, depth, accel, ms):
    from paper_2605_05543_amd import _lib

    print(f"case split precision={precision} n={n} depth={depth} accel={accel}", flush=True)
    dt = 1e-13
    orc = oracle.get()
    T, w, v = bunch.wiggly_history(n, depth, dt, beta=0.9, accel_rel=accel, seed=n + depth)
    rng = np.random.default_rng(n)
    with _lib.Context(n=n, depth=depth, q=Q, m=ME, dt=dt, precision=precision) as ctx:
        ctx.set_history(T, w, v, np.zeros((3, n)))
        for m in ms:
            x = 1.5e-3 * rng.standard_normal((3, m))
            si = np.full(m, -1, np.int64)
            x[:, 0], si[0] = w[-1][:, n // 2], n // 2  # on a source, excluded
            E, B, k = _fields(_lib.empp_fields_at_dev, ctx, T[-1], x, si)
            sub = np.unique(np.r_[0, m - 1, np.arange(0, m, max(1, m // 32))])
            E0, B0, k0, SE, SB = orc.fields(T, w, v, Q, T[-1], x[:, sub], si[sub], want_kstar=True, want_abs=True)
            (assert_mixed if precision else assert_fields)(f"m={m}", E[:, sub], B[:, sub], E0, B0, SE, SB)
            assert_kstar(f"m={m}", k[sub], k0)
            for fn, guess, want in ((_lib.empp_fields_at_dev, 0, False), (_lib.empp_fields_at_dev_noalloc, 0, True),
                                    (_lib.empp_fields_at_dev, 2, True)):
                ctx.set_mode(precision, guess)
                E2, B2, k2 = _fields(fn, ctx, T[-1], x, si, want)
                ctx.set_mode(precision, 0)
                assert np.array_equal(E, E2) and np.array_equal(B, B2), (m, guess, want)
                assert k2 is None or np.array_equal(k, k2), (m, guess)
