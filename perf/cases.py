"""Workloads that stand for what programs have this library do, for timing.

listed() names them, draw(rng) gives more of the same ranges, prepare() makes
what a program has in hand before the call (a context with its history, a
trained network, device buffers), run() is one pass through the public entry
points and returns its outputs, work() is what a pass cannot do without, and
exact() the same outputs in plain FP64 torch, without the library.

Sizes are those of the package's workloads (bunch.py), of its tests, or
between them; bunches are Gaussian (Sec. 2.5 of arXiv 2605.05543), and a
history spans about 50 ps (512 slots of 0.1 ps) whatever its depth.
"""
import math

import numpy as np
import torch

from paper_2605_05543_amd import _lib, bunch

C = bunch.C_LIGHT
Q, ME = -bunch.E_CHARGE, bunch.M_ELECTRON
MU0 = 1.25663706212e-6
KQ = Q * MU0 * C * C / (4.0 * math.pi)
SPAN = 512 * 1e-13  # seconds of stored history

PRECISION = {"fp64": _lib.EMPP_FP64, "mixed": _lib.EMPP_MIXED}
GUESS = {"bisect": _lib.EMPP_GUESS_BISECT, "straight": _lib.EMPP_GUESS_BALLISTIC, "network": _lib.EMPP_GUESS_MLP,
         "previous": _lib.EMPP_GUESS_PREVIOUS}


def _step(name, n, depth, *, precision="fp64", guess="bisect", steps=1, mev=1.0, dipole=False, adaptive=False,
          curved=False, group=0):
    return {"name": name, "kind": "step", "n": n, "depth": depth, "precision": precision, "guess": guess,
            "steps": steps, "mev": mev, "dipole": dipole, "adaptive": adaptive, "curved": curved, "group": group}


def _fields(name, m, n, depth, *, precision="fp64", guess="bisect", host=False, kstar=False, curved=False, mev=1.0):
    return {"name": name, "kind": "fields", "m": m, "n": n, "depth": depth, "precision": precision, "guess": guess,
            "host": host, "kstar": kstar, "curved": curved, "mev": mev}


def listed():
    return [
        # the smallest bunch (N = 256, D = 256): a short run of steps, then its
        # state is read: launches and latency count
        _step("step_n256_d256_x10", 256, 256, steps=10),
        # a field map: a few points outside the bunch, device buffers
        _fields("fields_m64_n8192_d512", 64, 8192, 512),
        # a checked field call from host arrays, ragged sizes, with the bracket
        # of every pair, on curving paths
        _fields("fields_host_m257_n1000_d129", 257, 1000, 129, guess="straight", host=True, kstar=True, curved=True),
        # the N = 8192 bunch: an ordinary step of the plain path
        _step("step_n8192_d512", 8192, 512, mev=2.0),
        # the same with the step size chosen on the device, a ragged bunch
        _step("step_n5000_d300_adaptive", 5000, 300, adaptive=True),
        # a bunch gyrating in a strong field: histories that curve
        _step("step_n16384_d512_curved", 16384, 512, curved=True),
        # warm-started brackets, several steps of a middle-sized bunch
        _step("step_n16384_d512_previous_x3", 16384, 512, guess="previous", steps=3),
        # the full-size bunch at 3 Earth radii, the plain FP64 path
        _step("step_n65536_d512_dipole", 65536, 512, dipole=True),
        # the same in mixed precision with the trained network's guesses
        _step("step_n65536_d512_mixed_network", 65536, 512, precision="mixed", guess="network", dipole=True,
              group=12),
        # a deep history at 5 MeV with the straight-line guess
        _step("step_n32768_d1024_straight", 32768, 1024, guess="straight", mev=5.0, dipole=True),
        # training of the delay network on device rows
        {"name": "train_b8192_x32", "kind": "train", "batch": 8192, "rows": 1 << 18, "steps": 32},
        # Stage II: transport in the dipole after the handoff
        {"name": "transport_n65536_x100", "kind": "transport", "n": 65536, "steps": 100},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "fields", "fields", "train", "transport"])
    if kind == "train":
        return {"kind": "train", "batch": 64 * _log_int(rng, 4, 128), "rows": _log_int(rng, 10000, 1 << 18),
                "steps": rng.randint(4, 32)}
    if kind == "transport":
        return {"kind": "transport", "n": _log_int(rng, 100, 65536), "steps": rng.randint(20, 100)}
    depth = _log_int(rng, 16, 1024)
    if kind == "fields":
        n = _log_int(rng, 64, 32768)
        host = rng.random() < 0.4
        c = _fields("", _log_int(rng, 1, 4096), n, depth, precision=rng.choice(["fp64", "fp64", "mixed"]),
                    guess=rng.choice(["bisect", "bisect", "straight"]), host=host,
                    kstar=host and n <= 8192 and rng.random() < 0.5, curved=n * depth < 4e6 and rng.random() < 0.3,
                    mev=rng.choice([1.0, 2.0, 5.0]))
        if c["kstar"]:
            c["m"] = min(c["m"], 512)
    else:
        n = _log_int(rng, 64, 32768)
        precision = rng.choice(["fp64", "fp64", "mixed"])
        guess = rng.choice(["bisect", "bisect", "straight", "network", "previous"])
        adaptive = rng.random() < 0.2
        if precision == "mixed" and guess == "previous":
            guess = "bisect"
        if adaptive:
            precision, guess = "fp64", rng.choice(["bisect", "straight", "previous"])
        curved = n * depth < 9e6 and rng.random() < 0.25
        c = _step("", n, depth, precision=precision, guess=guess, steps=rng.randint(1, 10) if n < 2048 else 1,
                  mev=rng.choice([1.0, 2.0, 5.0]), dipole=not curved and rng.random() < 0.5, adaptive=adaptive,
                  curved=curved,
                  group=rng.choice([0, 8, 12]) if guess == "network" else 0)
    del c["name"]
    return c


# -- inputs ---------------------------------------------------------------------


def _bunch(n, mev, seed, dipole=False):
    center = (3 * bunch.R_EARTH, 0.0, 0.0) if dipole else (0.0, 0.0, 0.0)
    return bunch.gaussian_bunch(bunch.BunchSpec(n, (1e-3, 1e-3, 1e-3), mev, center=center, seed=seed))


def _curved_history(case, seed):
    """A Gaussian bunch gyrating: 1.5 rad of turn over the stored history,
    every segment moving at its stored velocity."""
    n, depth = case["n"], case["depth"]
    dt = SPAN / depth
    r, u = _bunch(n, case["mev"], seed)
    u = bunch.beam_rotation(math.pi / 2, math.pi / 2) @ u
    gam = np.sqrt(1.0 + (u * u).sum(0) / C**2)
    vel = u / gam
    T = dt * np.arange(-(depth - 1), 1, dtype=np.float64)
    ang = (1.5 / SPAN) * T
    v = np.empty((depth, 3, n))
    for k in range(depth):
        ca, sa = math.cos(ang[k]), math.sin(ang[k])
        v[k, 0] = ca * vel[0] - sa * vel[1]
        v[k, 1] = sa * vel[0] + ca * vel[1]
        v[k, 2] = vel[2]
    w = np.empty((depth, 3, n))
    w[depth - 1] = r
    for k in range(depth - 2, -1, -1):
        w[k] = w[k + 1] - v[k] * (T[k + 1] - T[k])
    v[depth - 1] = v[depth - 2]  # provisional
    return T, w, v, np.ascontiguousarray(gam * v[depth - 1])


def _context(case, **more):
    dipole = bool(case.get("dipole", False))
    return _lib.Context(n=case["n"], depth=case["depth"], q=Q, m=ME, dt=SPAN / case["depth"], ext_field=int(dipole),
                        dipole_b0=bunch.C3.dipole_b0 if dipole else 0.0, dipole_re=bunch.R_EARTH if dipole else 0.0,
                        **more)


def _load(ctx, case, seed):
    if case.get("curved"):
        T, w, v, u = _curved_history(case, seed)
        ctx.set_history(T, w, v, u)
    else:
        r, u = _bunch(case["n"], case["mev"], seed, bool(case.get("dipole")))
        ctx.init_bunch(r, u, 0.0)
        ctx.init_history_straight()


def _train_network(ctx, case, seed):
    ctx.surrogate_set(bunch.surrogate_init(seed % 1000), 1e-3)
    X, y = ctx.surrogate_samples_torch(1 << 16, seed=seed)
    ctx.surrogate_train_torch(X, y, steps=100, batch=8192, lr=3e-3, lr_final=3e-5)


def _points(case, seed):
    """Targets of a field call: points about the bunch, a quarter of them on
    particles (which then leave themselves out)."""
    rng = np.random.default_rng([seed, 17])
    m, n = case["m"], case["n"]
    x = 1.5e-3 * rng.standard_normal((3, m))
    idx = np.full(m, -1, dtype=np.int64)
    own = rng.random(m) < 0.25
    idx[own] = rng.integers(0, n, int(own.sum()))
    return x, idx


def _positions(case, seed):
    return _curved_history(case, seed)[1][-1] if case.get("curved") else _bunch(case["n"], case["mev"], seed)[0]


def _targets(case, seed):
    x, idx = _points(case, seed)
    own = idx >= 0
    x[:, own] = _positions(case, seed)[:, idx[own]]
    return x, idx


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        ctx = _context(case, guess=GUESS["previous"] if case["guess"] == "previous" else 0,
                       adaptive=case["adaptive"], guess_group_log2=case["group"])
        _load(ctx, case, seed)
        if case["guess"] == "network":
            _train_network(ctx, case, seed)
        ctx.set_mode(PRECISION[case["precision"]], GUESS[case["guess"]])
        return {"case": case, "ctx": ctx}
    if kind == "fields":
        ctx = _context(case)
        _load(ctx, case, seed)
        ctx.set_mode(PRECISION[case["precision"]], GUESS[case["guess"]])
        x, idx = _targets(case, seed)
        s = {"case": case, "ctx": ctx, "x": x, "idx": idx}
        if not case["host"]:
            s["x"] = torch.tensor(x, device="cuda")
            s["idx"] = torch.tensor(idx, device="cuda")
            s["E"] = torch.empty((3, case["m"]), dtype=torch.float64, device="cuda")
            s["B"] = torch.empty_like(s["E"])
        return s
    if kind == "train":
        src = {"n": 2048, "depth": 64, "mev": 2.0, "curved": True}
        ctx = _context(src)
        _load(ctx, src, seed)
        ctx.surrogate_set(bunch.surrogate_init(seed % 1000), 1e-3)
        X, y = ctx.surrogate_samples_torch(case["rows"], seed=seed)
        return {"case": case, "ctx": ctx, "X": X, "y": y, "params": bunch.surrogate_init(seed % 1000)}
    if kind == "transport":
        ctx = _context({"n": case["n"], "depth": 2, "dipole": True})
        r, u = _bunch(case["n"], 1.0, seed, True)
        ctx.init_bunch(r, bunch.beam_rotation(math.pi / 6, 0.0) @ u, 0.0)
        ctx.init_history_straight()
        ctx.handoff()
        return {"case": case, "ctx": ctx}
    raise ValueError(kind)


# -- one pass -------------------------------------------------------------------

DT_MAX, GYRO = 1e-7, 1.0 / 32.0  # Stage II's largest step and its part of a gyro-period
LR, LR_FINAL = 3e-3, 3e-5


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "step":
        ctx.step(case["steps"])
        E, B = ctx.fields()
        r, u, t, _ = ctx.state()
        return {"E": E, "B": B, "r": r, "u": u, "t": t}
    if kind == "fields":
        if case["host"]:
            out = ctx.fields_at(0.0, s["x"], s["idx"], want_kstar=case["kstar"])
            return dict(zip(("E", "B", "kstar"), out))
        _lib.empp_fields_at_dev(ctx.h, 0.0, case["m"], s["x"].data_ptr(), s["idx"].data_ptr(), s["E"].data_ptr(),
                                s["B"].data_ptr())
        return {"E": s["E"], "B": s["B"]}
    if kind == "train":
        ctx.surrogate_set(s["params"], 1e-3)
        ctx.surrogate_train_torch(s["X"], s["y"], steps=case["steps"], batch=case["batch"], lr=LR, lr_final=LR_FINAL)
        return {"params": ctx.surrogate_get()}
    ctx.transport(DT_MAX, GYRO, case["steps"])
    r, u, t, _ = ctx.state()
    return {"r": r, "u": u, "t": t}


# operations of a pair: two sign tests (9 each), the root (32), the
# reconstruction (20), the fields (69) and their sum (6)
PAIR_FLOP = 2 * 9 + 32 + 20 + 69 + 6
NET_MACS = 10 * 128 + 128 * 128 + 128


def work(case):
    kind = case["kind"]
    if kind in ("step", "fields"):
        n, depth = case["n"], case["depth"]
        m = case["m"] if kind == "fields" else n
        steps = case.get("steps", 1)
        pairs = float(m) * n * steps
        # the stored positions and velocities once; targets in, fields out
        by = steps * (48.0 * n * depth + 72.0 * m)
        if kind == "step":
            by += steps * 144.0 * n  # proper velocities, the new slot
        if case.get("kstar"):
            by += 4.0 * m * n
        if case.get("guess") == "previous":
            by += 4.0 * n * n * steps
        return {"bytes": by, "flops": PAIR_FLOP * pairs}
    if kind == "train":
        rows = float(case["batch"]) * case["steps"]
        return {"bytes": 44.0 * rows + 18049 * 4 * 7.0 * case["steps"], "flops": 6.0 * NET_MACS * rows}
    n, k = float(case["n"]), case["steps"]
    return {"bytes": 96.0 * n * k, "flops": 120.0 * n * k}


# -- the same in plain FP64 torch -------------------------------------------------


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _pair_fields(T, wt, vt, x, idx, want_kstar=False, eta=None):
    """Fields at x[3, m] of sources with history wt, vt [N, D, 3] at times
    T[D] (oldest first), leaving out source idx[a] of target a.  eta: also
    (min |eta|, max |v_i - v_j(t_r)|) with the targets' velocities eta[m, 3]."""
    N, D, _ = wt.shape
    m = x.shape[1]
    dev = wt.device
    wf, vf = wt.reshape(N * D, 3), vt.reshape(N * D, 3)
    L = C * (T[-1] - T)
    inv_h = torch.cat([1.0 / (T[1:] - T[:-1]), torch.zeros(1, dtype=T.dtype, device=dev)])
    E = torch.empty((m, 3), dtype=torch.float64, device=dev)
    B = torch.empty_like(E)
    ks = torch.empty((m, N), dtype=torch.int32, device=dev) if want_kstar else None
    row = torch.arange(N, device=dev) * D
    emin, vmax = math.inf, 0.0
    step = max(1, (1 << 23) // N)
    for a0 in range(0, m, step):
        xa = x[:, a0:a0 + step].T[:, None, :]
        k = xa.shape[0]
        skip = torch.arange(N, device=dev)[None, :] == idx[a0:a0 + step, None]

        def inside(s):
            d = xa - wf[row + s]
            return L[s] ** 2 > (d * d).sum(-1)

        lo = torch.zeros((k, N), dtype=torch.int64, device=dev)
        before = ~inside(lo)
        hi = torch.full_like(lo, D - 1)
        for _ in range(max(1, math.ceil(math.log2(D)))):
            mid = (lo + hi) // 2
            ok = inside(mid)
            lo, hi = torch.where(ok, mid, lo), torch.where(ok, hi, mid)
        lo = torch.where(before, torch.zeros_like(lo), lo)
        if want_kstar:
            kk = torch.where(before, torch.full_like(lo, -1), D - 1 - lo)
            ks[a0:a0 + step] = torch.where(skip, torch.zeros_like(kk), kk).to(torch.int32)
        nx = torch.clamp(lo + 1, max=D - 1)
        v1, v2 = vf[row + lo], vf[row + nx]
        d, L1 = xa - wf[row + lo], L[lo]
        C2 = C * C - (v1 * v1).sum(-1)
        C1 = (d * v1).sum(-1) - C * L1
        C0 = L1 * L1 - (d * d).sum(-1)
        dt = C0 / (torch.sqrt(torch.clamp(C1 * C1 - C2 * C0, min=0.0)) - C1)
        a = (v2 - v1) * (inv_h[lo] * ~before)[..., None]
        vr = v1 + a * dt[..., None]
        e = d - v1 * dt[..., None]
        en = torch.where(skip, torch.ones_like(dt), L1 - C * dt)
        if eta is not None:
            use = ~skip
            dv = ((eta[a0:a0 + step, None, :] - vr) ** 2).sum(-1)
            emin, vmax = min(emin, float(en[use].min())), max(vmax, float(dv[use].max().sqrt()))
        ev = C * en - (e * vr).sum(-1)
        pv = C * e / en[..., None] - vr
        pref = torch.where(skip, torch.zeros_like(en), KQ * en / ev ** 3)
        Ep = pref[..., None] * (((C * C - (vr * vr).sum(-1)) + (e * a).sum(-1))[..., None] * pv - ev[..., None] * a)
        Ep = torch.where(skip[..., None], torch.zeros_like(Ep), Ep)
        E[a0:a0 + step] = Ep.sum(1)
        B[a0:a0 + step] = torch.linalg.cross(e / (C * en)[..., None], Ep).sum(1)
    return E.T, B.T, ks, emin, vmax


def _dipole(x, k):
    r = x.norm(dim=0)
    mr = x[2] / r
    b = 3.0 * mr * x / r
    b[2] = b[2] - 1.0
    return k / r ** 3 * b


def _higuera_cary(u, E, B, eps):
    um = u + eps * E
    t = eps * B
    g2 = 1.0 + (um * um).sum(0) / C**2
    us = (um * t).sum(0) / C
    tau2 = (t * t).sum(0)
    sg = g2 - tau2
    t = t / torch.sqrt(0.5 * (sg + torch.sqrt(sg * sg + 4.0 * (tau2 + us * us))))
    up = (um + (um * t).sum(0) * t + torch.linalg.cross(um, t, dim=0)) / (1.0 + (t * t).sum(0))
    return up + eps * E + torch.linalg.cross(up, t, dim=0)


def _history(case, seed, dev):
    if case.get("curved"):
        T, w, v, u = (torch.tensor(a, device=dev) for a in _curved_history(case, seed))
        return T, w.permute(2, 0, 1).contiguous(), v.permute(2, 0, 1).contiguous(), u
    r, u = (torch.tensor(a, device=dev) for a in _bunch(case["n"], case["mev"], seed, bool(case.get("dipole"))))
    depth = case["depth"]
    v0 = u / torch.sqrt(1.0 + (u * u).sum(0) / C**2)
    T = (SPAN / depth) * torch.arange(-(depth - 1), 1, dtype=torch.float64, device=dev)
    w = r.T[:, None, :] + v0.T[:, None, :] * T[None, :, None]
    return T, w.contiguous(), v0.T[:, None, :].expand(-1, depth, -1).contiguous(), u


def _exact_step(case, seed):
    dev = _dev()
    T, w, v, u = _history(case, seed, dev)
    n, dt0 = case["n"], SPAN / case["depth"]
    idx = torch.arange(n, device=dev)
    dip = bunch.C3.dipole_b0 * bunch.R_EARTH**3
    t0 = float(T[-1])
    for k in range(case["steps"]):
        x = w[:, -1, :].T.contiguous()
        E, B, _, emin, vmax = _pair_fields(T, w, v, x, idx, eta=v[:, -1, :] if case["adaptive"] else None)
        dt = dt0
        if case["adaptive"]:
            dt = min(1e-12, max(1e-15, 0.05 * emin / vmax))
        Bt = B + _dipole(x, dip) if case["dipole"] else B
        u = _higuera_cary(u, E, Bt, Q * dt / (2.0 * ME))
        vn = u / torch.sqrt(1.0 + (u * u).sum(0) / C**2)
        tn = float(T[-1]) + dt if case["adaptive"] else t0 + (k + 1) * dt0
        v[:, -1, :] = vn.T
        w = torch.cat([w[:, 1:], (x + vn * dt).T[:, None, :]], 1)
        v = torch.cat([v[:, 1:], vn.T[:, None, :]], 1)
        T = torch.cat([T[1:], torch.tensor([tn], dtype=torch.float64, device=dev)])
    return {"E": E, "B": B, "r": w[:, -1, :].T.contiguous(), "u": u, "t": float(T[-1])}


def _exact_fields(case, seed):
    dev = _dev()
    T, w, v, _ = _history(case, seed, dev)
    x, idx = (torch.tensor(a, device=dev) for a in _targets(case, seed))
    E, B, ks, _, _ = _pair_fields(T, w, v, x, idx, want_kstar=case["kstar"])
    out = {"E": E, "B": B}
    if case["kstar"]:
        out["kstar"] = ks
    return out


def _exact_transport(case, seed):
    dev = _dev()
    r, u = _bunch(case["n"], 1.0, seed, True)
    x, u = torch.tensor(r, device=dev), torch.tensor(bunch.beam_rotation(math.pi / 6, 0.0) @ u, device=dev)
    dip, t = bunch.C3.dipole_b0 * bunch.R_EARTH**3, 0.0
    for _ in range(case["steps"]):
        B = _dipole(x, dip)
        g = torch.sqrt(1.0 + (u * u).sum(0) / C**2)
        dt = min(DT_MAX, GYRO * 2.0 * math.pi * ME / abs(Q) * float((g / B.norm(dim=0)).min()))
        u = _higuera_cary(u, torch.zeros_like(u), B, Q * dt / (2.0 * ME))
        x = x + u / torch.sqrt(1.0 + (u * u).sum(0) / C**2) * dt
        t += dt
    return {"r": x, "u": u, "t": t}


def exact(case, seed):
    if case["kind"] == "step":
        return _exact_step(case, seed)
    if case["kind"] == "fields":
        return _exact_fields(case, seed)
    if case["kind"] == "transport":
        return _exact_transport(case, seed)
    # the trained weights: the optimiser amplifies the rounding of bf16
    # activations, so plain FP64 training ends elsewhere
    return None
