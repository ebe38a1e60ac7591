"""Training launches at the edges of their blocks of 64 rows against the FP64
oracle: one row to more rows than resident blocks hold at once, batches whose
launch has blocks without rows, and several barriers in a row.  Tolerances:
gradient 3e-2 relative (a few bfloat16 roundings of 2^-9 in a chain of three
layers, as for the parts of the gradient elsewhere), Adam 1e-6 (float32)."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2605_05543_amd import bunch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 63, 65, 640, 8192, 8256, 20000])
def test_training_blocks(rows):
    import torch

    from paper_2605_05543_amd._lib import Context

    print(f"case training blocks rows={rows}", flush=True)
    rng = np.random.default_rng(rows)
    P = bunch.surrogate_init(3)
    X = rng.standard_normal((rows, 10)).astype(np.float32)
    X[:, 3:9] *= 0.5
    y = rng.standard_normal(rows).astype(np.float32)
    batch = rows // 64 * 64
    with Context(n=8, depth=8, q=-bunch.E_CHARGE, m=bunch.M_ELECTRON, dt=1e-13) as ctx:
        ctx.surrogate_set(P, 1e-3)
        loss, g = ctx.surrogate_loss_grad(X, y)
        lo, go = omlp.loss_and_grad(P.astype(np.float64), X.astype(np.float64), y.astype(np.float64))
        err = np.linalg.norm(g - go) / np.linalg.norm(go)
        print(f"   loss {abs(loss - lo) / lo:.1e}, gradient {err:.1e}", flush=True)
        assert abs(loss - lo) < 3e-2 * lo and err < 3e-2
        if batch == 0:
            return
        _, gb = ctx.surrogate_loss_grad(X[:batch], y[:batch])
        Xt, yt = torch.tensor(X[:batch], device="cuda"), torch.tensor(y[:batch], device="cuda")
        # one step from the launch's own gradient; the second's from the first's weights
        m = v = 0.0
        Po = P.astype(np.float64)
        for k in (1, 2):
            ctx.surrogate_train_torch(Xt, yt, steps=1, batch=batch, lr=1e-3, lr_final=1e-3)
            P1 = ctx.surrogate_get()
            Po, m, v = omlp.adam_step(Po, m, v, gb.astype(np.float64), k, 1e-3)
            assert np.max(np.abs(P1 - Po)) < 1e-6, k
            _, gb = ctx.surrogate_loss_grad(X[:batch], y[:batch])
        ctx.surrogate_set(P, 1e-3)
        ctx.surrogate_train_torch(Xt, yt, steps=2, batch=batch, lr=1e-3, lr_final=1e-3)
        assert np.array_equal(ctx.surrogate_get(), P1)  # both steps in one launch
