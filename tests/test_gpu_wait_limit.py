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


@pytest.mark.parametrize("steps", [8, 300])
def test_training_that_gives_up(steps):
    import torch

    print(f"case training gives up steps={steps}", flush=True)
    P = bunch.surrogate_init(2)
    rng = np.random.default_rng(3)
    X = rng.standard_normal((8192, 10)).astype(np.float32)
    y = rng.standard_normal(8192).astype(np.float32)
    Xt, yt = torch.tensor(X, device="cuda"), torch.tensor(y, device="cuda")
    kw = dict(n=8, depth=8, q=Q, m=ME, dt=1e-13)

    def run(ctx):
        ctx.surrogate_set(P, 1e-3)
        ctx.surrogate_train_torch(Xt, yt, steps=20, batch=4096, lr=1e-3, lr_final=1e-4)
        return ctx.surrogate_get()

    with _lib.Context(**kw) as ctx:
        ref = run(ctx)
    with _lib.Context(**kw) as ctx:
        run(ctx)
        _wait_polls(ctx, 0)
        with pytest.raises(_lib.EmppError) as ei:
            ctx.surrogate_loss_grad(X, y)
        assert ei.value.status == _lib.EMPP_EDEVICE
        assert np.array_equal(ctx.surrogate_get(), ref)  # an evaluation leaves the network
        with pytest.raises(_lib.EmppError) as ei:
            ctx.surrogate_train_torch(Xt, yt, steps=steps, batch=4096, lr=1e-3, lr_final=1e-4)
        assert ei.value.status == _lib.EMPP_EDEVICE
        _wait_polls(ctx, 1 << 24)
        for call in (ctx.surrogate_get, lambda: ctx.surrogate_loss_grad(X, y),
                     lambda: ctx.surrogate_train_torch(Xt, yt, steps=2, batch=4096, lr=1e-3, lr_final=1e-4)):
            with pytest.raises(_lib.EmppError) as ei:
                call()
            assert ei.value.status == _lib.EMPP_ESTATE
        assert np.array_equal(run(ctx), ref)


def test_training_beside_a_stepping_context():
    """A thread that trains small batches on a stream of its own while another
    steps a bunch whose pair passes fill the chip: each ends where it ends alone."""
    import threading

    import torch

    print("case training beside steps", flush=True)
    P = bunch.surrogate_init(2)
    rng = np.random.default_rng(3)
    X = rng.standard_normal((4096, 10)).astype(np.float32)
    y = rng.standard_normal(4096).astype(np.float32)
    r, ub = bunch.gaussian_bunch(bunch.BunchSpec(16384, (1e-3, 1e-3, 1e-3), 1.0, seed=3))

    def run(kind, out, i):
        with torch.cuda.stream(torch.cuda.Stream()):
            if kind == "step":
                with _lib.Context(n=16384, depth=64, q=Q, m=ME, dt=1e-13) as ctx:
                    ctx.init_bunch(r, ub, 0.0)
                    ctx.init_history_straight()
                    for _ in range(30):
                        ctx.step(2)
                        E, B = ctx.fields()
                    out[i] = (E, B, *ctx.state()[:2])
            else:
                Xt, yt = torch.tensor(X, device="cuda"), torch.tensor(y, device="cuda")
                with _lib.Context(n=8, depth=8, q=Q, m=ME, dt=1e-13) as ctx:
                    ctx.surrogate_set(P, 1e-3)
                    for _ in range(20):
                        ctx.surrogate_train_torch(Xt, yt, steps=20, batch=256, lr=1e-3, lr_final=1e-4)
                    out[i] = (ctx.surrogate_get(),)

    kinds = ["train", "step", "train"]
    alone, beside = [None] * 3, [None] * 3
    for i, k in enumerate(kinds):
        run(k, alone, i)
    threads = [threading.Thread(target=run, args=(k, beside, i)) for i, k in enumerate(kinds)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    for a, b in zip(alone, beside):
        assert b is not None and all(np.array_equal(x, z) for x, z in zip(a, b))
