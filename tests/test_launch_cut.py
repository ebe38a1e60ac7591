"""The cut of a pair launch fits the partials its context holds, for every
search mode and precision a context can be switched to: the layout is made once,
with the mode at creation.  Host arithmetic only (no GPU)."""
import ctypes

import pytest

from paper_2605_05543_amd import _lib, bunch

Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON
MODES = [(_lib.EMPP_FP64, g) for g in (0, 1, 2, 3, 4)] + [(_lib.EMPP_MIXED, g) for g in (0, 1, 2, 3)]


def _cut(cfg, precision, guess, m):
    out = (ctypes.c_int64 * 6)()
    st = _lib.lib.empp_internal_launch_cut(ctypes.byref(cfg), precision, guess, ctypes.c_int64(m), out)
    assert st == _lib.EMPP_OK
    return dict(zip(("chunks", "src", "sg", "held", "nominal", "most"), out))


@pytest.mark.parametrize("created", [0, 2, 4])
@pytest.mark.parametrize("splits", [0, 1, 37, 2000])
def test_cut_fits_the_partials(created, splits):
    sizes = [2, 3, 64, 65, 1000, 8192, 16385, 29184, 33280, 50000, 65536, 100000, 140000, 200000, 262144, 1 << 20]
    for n in sizes:
        for depth in (5, 512, 1024, 3000):
            cfg = _lib.Config(n=n, depth=depth, q=Q, m=ME, dt=1e-13, guess=created, source_splits=splits)
            for precision, guess in MODES:
                if guess == 4 and created != 4:
                    continue
                ms = {1, 63, 65, 1025, n // 3, n // 2 + 1, n - 1, n, 2 * n}
                for m in sorted(x for x in ms if x >= 1):
                    c = _cut(cfg, precision, guess, m)
                    at = (n, depth, precision, guess, m, c)
                    launched = min(m, n)
                    assert 1 <= c["chunks"] and (c["chunks"] - 1) * c["src"] < n <= c["chunks"] * c["src"], at
                    assert c["chunks"] * launched <= c["held"] * n, at
                    assert precision == _lib.EMPP_FP64 or c["sg"] == 0, at
                    if m <= c["most"]:  # the allocation-free call's 128 MiB
                        assert c["chunks"] * launched * 96 <= 128 << 20, at


def test_fp64_modes_of_a_context_share_the_cut():
    """So that they add in the same order: fields are bit-identical."""
    for n, depth in ((1000, 64), (65536, 512), (100000, 1024)):
        for created in (0, 4):
            cfg = _lib.Config(n=n, depth=depth, q=Q, m=ME, dt=1e-13, guess=created)
            for m in (65, n):
                cuts = [_cut(cfg, _lib.EMPP_FP64, g, m) for g in ((0, 1, 2, 3, 4) if created == 4 else (0, 1, 2, 3))]
                assert all(c == cuts[0] for c in cuts)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
def test_switched_context_against_the_oracle(precision):
    """A warm-start context switched to another mode, at a size whose launches in
    that mode take more chunks where the layout allows them.  Tolerances: those of
    every field (parity.FP64_TOL, parity.MIXED_TOL)."""
    import numpy as np

    import oracle
    from parity import assert_fields, assert_mixed
    from test_zz_no_alloc import _fields

    n, depth, dt = 50000, 4, 1e-13
    print(f"case switched context precision={precision}", flush=True)
    orc = oracle.get()
    r, u = bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), 1.0, seed=6))
    T, w, v = orc.init_straight(r, u, depth, dt)
    sub = bunch.target_subset(n, 64, 9)
    E0, B0, SE, SB = orc.fields(T, w, v, Q, T[-1], r[:, sub], sub, want_abs=True)
    check = assert_mixed if precision else assert_fields
    with _lib.Context(n=n, depth=depth, q=Q, m=ME, dt=dt, guess=_lib.EMPP_GUESS_PREVIOUS) as ctx:
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()
        for guess in (0, 2):
            ctx.set_mode(precision, guess)
            for fn in (_lib.empp_fields_at_dev, _lib.empp_fields_at_dev_noalloc):
                m = 15000
                x, idx = r.copy()[:, :m], np.arange(m)
                x[:, :64], idx[:64] = r[:, sub], sub
                E, B, _ = _fields(fn, ctx, 0.0, x, idx, want_kstar=False)
                check(f"fields guess={guess}", E[:, :64], B[:, :64], E0, B0, SE, SB)
        ctx.step(1)
        E, B = ctx.fields()
        check("step", E[:, sub], B[:, sub], E0, B0, SE, SB)
        ctx.set_mode(0, _lib.EMPP_GUESS_PREVIOUS)
        ctx.step(2)
        assert np.all(np.isfinite(ctx.fields()[0]))
