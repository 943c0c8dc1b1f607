"""Curvilinear pipelines: rollouts of few samples give the bits of the one-wave rollout
(the first samples of a problem large enough for it), and the adjoint that stores every
state agrees with the oracle's dual-number gradient."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep
from test_gpu_adjoint import OBJ_COST, OBJ_MIXED, _check_grad

pytestmark = pytest.mark.gpu


def _setup(shapes, dtype):
    f32 = dtype == torch.float32
    f = (lambda a: np.asarray(a, np.float32).astype(np.float64)) if f32 else np.asarray
    probs, tabs, x0s = [], [], []
    for b, (K, T) in enumerate(shapes):
        tr = W.spline_track(T)
        probs.append(W.Problem(K=K, T=T, track=tr, x0=W.start_state(tr),
                               V=W.test_sequences(1, T, seed=T, scale=0.4)[0], it=T))
        kappa, ds = W.curvature_table(tr)
        tabs.append((f(kappa), float(f(ds))))
        x0s.append(f(W.start_state_c8(vx=2.0 + 0.1 * b, e_y=0.2 - 0.05 * b, e_psi=0.1, s=93.0 + b)))
    probs = prep(probs, dtype)
    db = core.DeviceBatch(probs, dtype=dtype)
    ct = core.CurvTrackArrays(tabs, [p.track.half_width for p in probs], dtype=dtype)
    x0 = torch.as_tensor(np.concatenate(x0s), dtype=dtype, device="cuda")
    return probs, tabs, x0s, db, ct, x0, (W.wheels_f32() if f32 else W.WHEELS)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("T,Ks", [(1, (1,)), (2, (63,)), (3, (64,)), (4, (65,)), (9, (130,)), (33, (1000, 20000))])
def test_pipelined_curvilinear_rollout_is_bit_identical(T, Ks, dtype):
    M, C = params(dtype)

    def run(K):
        _, _, _, db, ct, x0, wh = _setup([(K, T)], dtype)
        return core.rollout_curvilinear(ctx(), db, ct, M, wh, C, 5, x0=x0, want_eps=True)

    S, eps = run(131072)
    for K in Ks:
        s, e = run(K)
        assert torch.equal(s, S[:K]) and torch.equal(e, eps[:K])
    assert ctx().device_errors() == 0


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-9), (torch.float32, 1e-3)])
def test_stored_curvilinear_adjoint_vs_oracle(dtype, tol):
    M, C = params(dtype)
    shapes = [(1, 1), (63, 2), (64, 3), (65, 4), (130, 5), (200, 9), (129, 17)]
    probs, tabs, x0s, db, ct, x0, wh = _setup(shapes, dtype)
    rng = np.random.default_rng(8)
    gs = [np.where(rng.random(p.K) < 8.0 / p.K, rng.uniform(-1, 1, p.K), 0.0) for p in probs]
    gs[4][:64] = 0.0  # a group of 64 without upstream gradient
    gs[4][100] = 1.0
    gs[5][:] = 0.0  # a problem without any
    if dtype == torch.float32:
        gs = [g.astype(np.float32).astype(np.float64) for g in gs]
    sig = np.array(C["sigma"])
    for obj in (OBJ_COST, OBJ_MIXED):
        out = core.rollout_backward_curvilinear(
            ctx(), db, ct, M, wh, C, 11, torch.as_tensor(np.concatenate(gs), dtype=dtype, device="cuda"), obj, x0=x0)
        for b, got in enumerate(db.controls(out)):
            p = probs[b]
            ref = np.zeros((p.T, 2))
            for m in np.nonzero(gs[b])[0]:
                eps = oracle.normals(11, b, p.it, int(m), p.T) * sig
                ref += gs[b][m] * oracle.gradient_dual_c8(M, wh, C, *tabs[b], p.track.half_width, x0s[b], p.V, obj, eps)
            if b == 5:
                assert not got.any()
            else:
                _check_grad(got, ref, tol, (b, shapes[b], obj))
    assert ctx().device_errors() == 0
