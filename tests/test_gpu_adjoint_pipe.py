"""The adjoint that stores every state (small scratch): horizons around its ring depths,
ragged sample groups, groups without upstream gradient, obstacles; and its agreement
with the checkpointed adjoint that larger batches take."""
import numpy as np
import pytest
import torch

from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep
from test_gpu_adjoint import OBJ_COST, OBJ_MIXED, _check_grad, _oracle_grad_sums

pytestmark = pytest.mark.gpu


def _problem(b, K, T, n_obs, kind="spline"):
    tr = W.circle_track() if kind == "circle" else W.spline_track(b)
    if n_obs:
        tr.obs = W.obstacles(tr, b, n_obs, keep_clear=1.0)
    V = W.test_sequences(1, T, seed=60 + b, scale=0.5)[0]
    return W.Problem(K=K, T=T, track=tr, x0=W.start_state(tr, vx=2.0 + 0.2 * b), V=V, pid=b, it=b)


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-9), (torch.float32, 1e-3)])
@pytest.mark.parametrize("n_obs", [0, 7])
def test_stored_adjoint_vs_oracle(n_obs, dtype, tol):
    M, C = params(dtype)
    shapes = [(1, 1), (63, 2), (64, 3), (65, 4), (70, 5), (130, 8), (200, 9), (129, 17)]
    probs = prep([_problem(b, K, T, n_obs, "circle" if b == 4 and not n_obs else "spline")
                  for b, (K, T) in enumerate(shapes)], dtype)
    db = core.DeviceBatch(probs, dtype=dtype)
    rng = np.random.default_rng(5)
    gs = [np.where(rng.random(p.K) < 12.0 / p.K, rng.uniform(-1, 1, p.K), 0.0) for p in probs]
    gs[5][:64] = 0.0  # a group of 64 without upstream gradient
    gs[5][100] = 1.0
    gs[6][:] = 0.0  # a problem without any
    if dtype == torch.float32:
        gs = [g.astype(np.float32).astype(np.float64) for g in gs]
    for obj in (OBJ_COST, OBJ_MIXED):
        out = core.rollout_backward(ctx(), db, M, C, 11, torch.as_tensor(np.concatenate(gs), dtype=dtype, device="cuda"),
                                    obj)
        ref, _ = _oracle_grad_sums(M, C, probs, 11, gs, obj)
        for b, got in enumerate(db.controls(out)):
            if b == 6:
                assert not got.any()
            else:
                _check_grad(got, ref[b], tol, (b, shapes[b], obj))
    assert ctx().device_errors() == 0


def test_zero_upstream_hides_a_diverged_sample():
    M, C = params(torch.float32)
    p = prep([_problem(0, 65, 6, 0)], torch.float32)[0]
    p.V[0, 0] = np.nan  # every sample of the problem diverges
    db = core.DeviceBatch([p])
    assert not core.rollout_backward(ctx(), db, M, C, 1, torch.zeros(65, device="cuda"), OBJ_COST).any()


@pytest.mark.parametrize("n_obs", [0, 64])
def test_stored_and_checkpointed_adjoints_agree(n_obs):
    """K = 65536, T = 100: every state fits the context's scratch (238 MB), checkpoints the
    fixed one (64 MB).  Both are FP32 sums of 65536 terms of about 100 chained steps, a few
    1e-6 from the FP64 gradient each."""
    M, C = params(torch.float32)
    p = prep([_problem(0, 65536, 100, n_obs)], torch.float32)[0]
    db = core.DeviceBatch([p])
    g = torch.rand(p.K, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    a = core.rollout_backward(ctx(), db, M, C, 3, g, OBJ_COST)
    b = core.rollout_backward(ctx(), db, M, C, 3, g, OBJ_COST, noalloc=True)
    assert (a - b).norm() <= 5e-5 * b.norm()
    assert ctx().device_errors() == 0
