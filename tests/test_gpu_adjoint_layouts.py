"""Both layouts of the adjoints, every state stored and checkpoints (what a ctx holds that was
reserved for less than the states), against the oracle's dual-number gradients at the same
small ragged shapes; and diverged samples without upstream gradient beside live ones."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2302_11719_amd import _lib as L
from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep
from test_gpu_adjoint import OBJ_COST, OBJ_MIXED, _check_grad, _oracle_grad_sums

pytestmark = pytest.mark.gpu
# K = 0 and 1, the edges of a group of 64 and ragged ones; horizons around the checkpoint
# segments (7 of the longest horizon's 37 steps)
SHAPES = [(1, 1), (63, 6), (64, 7), (65, 8), (0, 5), (300, 36), (129, 37), (257, 15)]


def _context(db, layout):
    """A ctx that holds the states of the batch, or (a sixth of its groups reserved) only
    its checkpoints."""
    if layout == "stored":
        return ctx()
    c = core.Context(0)
    groups = db.B * ((db.k_max + 63) // 64)
    bounds = L.Batch.from_buffer_copy(bytes(db.batch))
    bounds.n_problems, bounds.k_max = 1, 64 * (groups // 6)
    assert L.lib().smppi_reserve_batch(c.h, ctypes.byref(bounds)) == 0
    c.reserve = lambda _: None
    return c


def _upstream(probs, dtype, seed):
    rng = np.random.default_rng(seed)
    gs = []
    for p in probs:
        g = np.where(rng.random(p.K) < 8.0 / max(p.K, 1), rng.uniform(-1, 1, p.K), 0.0)
        if p.K:
            g[-1] = 1.0
        gs.append(g)
    gs[5][64:128] = 0.0  # a group of 64 without upstream gradient
    if dtype == torch.float32:
        gs = [g.astype(np.float32).astype(np.float64) for g in gs]
    return gs, torch.as_tensor(np.concatenate(gs), dtype=dtype, device="cuda")


def _run_both(db, call, check):
    out = {}
    for layout in ("stored", "checkpoints"):
        c = _context(db, layout)
        print(f"{db.dtype} {layout}", flush=True)
        out[layout] = call(c)
        assert c.device_errors() == 0
        for b, got in enumerate(db.controls(out[layout])):
            check(b, got, layout)
        if layout == "checkpoints":
            c.close()
    # (two orders of rounding: equal bits would mean that one layout ran twice)
    assert not torch.equal(out["stored"], out["checkpoints"])


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-9), (torch.float32, 1e-3)])
@pytest.mark.parametrize("n_obs,window,kind", [(0, 4, "spline"), (0, 7, "spline"), (0, 4, "circle"), (7, 4, "spline")])
def test_cartesian_layouts_vs_oracle(n_obs, window, kind, dtype, tol):
    M, C = params(dtype)
    probs = []
    for b, (K, T) in enumerate(SHAPES):
        tr = W.circle_track() if kind == "circle" else W.spline_track(b)
        tr.window = window
        if n_obs and b % 3 != 2:
            tr.obs = W.obstacles(tr, b, n_obs, keep_clear=1.0)
        V = W.test_sequences(1, T, seed=60 + b, scale=0.5)[0]
        probs.append(W.Problem(K=K, T=T, track=tr, x0=W.start_state(tr, vx=2.0 + 0.2 * b), V=V, pid=b, it=b))
    probs = prep(probs, dtype)
    db = core.DeviceBatch(probs, dtype=dtype)
    gs, g = _upstream(probs, dtype, 5)
    for obj in (OBJ_COST, OBJ_MIXED):
        ref, _ = _oracle_grad_sums(M, C, probs, 11, gs, obj)

        def check(b, got, layout):
            if probs[b].K:
                _check_grad(got, ref[b], tol, (layout, b, SHAPES[b], obj))
            else:
                assert not got.any()

        _run_both(db, lambda c: core.rollout_backward(c, db, M, C, 11, g, obj), check)


def _curvilinear(shapes, dtype):
    f32 = dtype == torch.float32
    f = (lambda a: np.asarray(a, np.float32).astype(np.float64)) if f32 else np.asarray
    probs, tabs, x0s = [], [], []
    for b, (K, T) in enumerate(shapes):
        tr = W.spline_track(b)
        probs.append(W.Problem(K=K, T=T, track=tr, x0=W.start_state(tr),
                               V=W.test_sequences(1, T, seed=60 + b, scale=0.4)[0], it=b))
        kappa, ds = W.curvature_table(tr)
        tabs.append((f(kappa), float(f(ds))))
        x0s.append(f(W.start_state_c8(vx=2.0 + 0.1 * b, e_y=0.2 - 0.05 * b, e_psi=0.1, s=93.0 + b)))
    probs = prep(probs, dtype)
    db = core.DeviceBatch(probs, dtype=dtype)
    ct = core.CurvTrackArrays(tabs, [p.track.half_width for p in probs], dtype=dtype)
    x0 = torch.as_tensor(np.concatenate(x0s), dtype=dtype, device="cuda")
    return probs, tabs, x0s, db, ct, x0, (W.wheels_f32() if f32 else W.WHEELS)


def _curvilinear_ref(M, wh, C, probs, tabs, x0s, gs, obj):
    sig = np.array(C["sigma"])
    out = []
    for b, p in enumerate(probs):
        ref = np.zeros((p.T, 2))
        for m in np.nonzero(gs[b])[0]:
            eps = oracle.normals(11, b, p.it, int(m), p.T) * sig
            ref += gs[b][m] * oracle.gradient_dual_c8(M, wh, C, *tabs[b], p.track.half_width, x0s[b], p.V, obj, eps)
        out.append(ref)
    return out


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-9), (torch.float32, 1e-3)])
def test_curvilinear_layouts_vs_oracle(dtype, tol):
    M, C = params(dtype)
    probs, tabs, x0s, db, ct, x0, wh = _curvilinear(SHAPES, dtype)
    gs, g = _upstream(probs, dtype, 8)
    for obj in (OBJ_COST, OBJ_MIXED):
        ref = _curvilinear_ref(M, wh, C, probs, tabs, x0s, gs, obj)

        def check(b, got, layout):
            if probs[b].K:
                _check_grad(got, ref[b], tol, (layout, b, SHAPES[b], obj))
            else:
                assert not got.any()

        _run_both(db, lambda c: core.rollout_backward_curvilinear(c, db, ct, M, wh, C, 11, g, obj, x0=x0), check)


@pytest.mark.parametrize("layout", ["stored", "checkpoints"])
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-9), (torch.float32, 1e-3)])
@pytest.mark.parametrize("model,n_obs", [("cartesian", 0), ("cartesian", 7), ("curvilinear", 0)])
def test_diverged_samples_without_upstream_in_a_live_group(model, n_obs, dtype, tol, layout):
    """A throttle noise that overflows the costs of every sample with one negative draw (a
    sample survives four steps with probability 1/16, its throttle on the upper bound).  The
    live samples have upstream gradient, the diverged ones of the same groups have none."""
    M, C = params(dtype)
    M, C = dict(M), dict(C)
    big = 1e25 if dtype == torch.float32 else 1.2e154
    C["sigma"] = (C["sigma"][0], big)
    M["u_lo"] = (M["u_lo"][0], -1e4 * big)
    shapes = [(1500, 4)] * 7  # (many groups, so that the states outgrow a small reservation)
    if model == "curvilinear":
        probs, tabs, x0s, db, ct, x0, wh = _curvilinear(shapes, dtype)
        S = core.rollout_curvilinear(ctx(), db, ct, M, wh, C, 11, x0=x0)
    else:
        probs = []
        for b, (K, T) in enumerate(shapes):
            tr = W.spline_track(b)
            if n_obs:
                tr.obs = W.obstacles(tr, b, n_obs, keep_clear=1.0)
            probs.append(W.Problem(K=K, T=T, track=tr, x0=W.start_state(tr, vx=3.0),
                                   V=W.test_sequences(1, T, seed=60 + b, scale=0.3)[0], pid=b, it=b))
        probs = prep(probs, dtype)
        db = core.DeviceBatch(probs, dtype=dtype)
        S = core.rollout(ctx(), db, M, C, 11)
    gs = []
    for p, s in zip(probs, db.per_problem(S)):
        live = s < 1e6
        # diverged samples in every full group of 64, live ones in most
        assert (~np.isfinite(s[:1472])).reshape(-1, 64).any(1).all()
        assert live[:1472].reshape(-1, 64).any(1).sum() > 18
        g = np.zeros(p.K)
        g[np.nonzero(live)[0][::6]] = 1.0
        gs.append(g)
    g = torch.as_tensor(np.concatenate(gs), dtype=dtype, device="cuda")
    c = _context(db, layout)
    if model == "curvilinear":
        out = core.rollout_backward_curvilinear(c, db, ct, M, wh, C, 11, g, OBJ_COST, x0=x0)
        ref = _curvilinear_ref(M, wh, C, probs, tabs, x0s, gs, OBJ_COST)
    else:
        out = core.rollout_backward(c, db, M, C, 11, g, OBJ_COST)
        ref, _ = _oracle_grad_sums(M, C, probs, 11, gs, OBJ_COST)
    for b, got in enumerate(db.controls(out)):
        _check_grad(got, ref[b], tol, (layout, b))
    assert c.device_errors() == 0
