"""Shield steps with Jacobian rows computed ahead on a fourth wave (ten steps at a time)
and obstacle gradients split over lanes: horizons at the edges of those chunks against the
oracle, and a batch larger than the card (three waves) gives the bits of a small one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep

pytestmark = pytest.mark.gpu

HORIZONS = (1, 2, 4, 5, 9, 14, 15, 16, 24, 25, 26)


def _problem(T, n_obs, pid=0):
    if n_obs:
        p = W.config4(K=1, T=T, n_obs=n_obs)
    else:
        tr = W.spline_track(T)
        p = W.Problem(1, T, tr, W.start_state(tr, vx=3.0 + 0.1 * T), None, pid, 0)
    p.V = W.test_sequences(1, T, seed=T, scale=0.8)[0]
    return p


@pytest.mark.parametrize("n_obs", [0, 1, 6, 64])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_shield_steps_vs_oracle(dtype, n_obs):
    """Ten steps of Algorithm 1; the tolerances are those of the shield's parity test."""
    probs = prep([_problem(T, n_obs) for T in HORIZONS], dtype)
    M, C = params(dtype)
    db = core.DeviceBatch(probs, dtype=dtype)
    got = db.controls(core.shield_repair(ctx(), db, M, C, db.V, 10, 0.05, W.OBJ_SHIELD))
    assert ctx().device_errors() == 0
    for p, g in zip(probs, got):
        ref = oracle.repair(M, C, p.track, p.x0, p.V, 10, 0.05, W.OBJ_SHIELD)
        tol = 1e-3 * max(np.linalg.norm(p.V), 1.0) if dtype == torch.float32 else 1e-9
        assert np.abs(g - ref).max() <= tol, (p.T, np.abs(g - ref).max())


def test_three_and_four_waves_give_the_same_bits():
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    one = [_problem(T, 0) for T in HORIZONS]
    many = [one[i % len(one)] for i in range(n_cu + len(one))]
    M, C = params(torch.float32)
    out = []
    for probs in (one, many):
        db = core.DeviceBatch(prep(probs, torch.float32), dtype=torch.float32)
        out.append(db.controls(core.shield_repair(ctx(), db, M, C, db.V, 10, 0.05, W.OBJ_SHIELD)))
    for i, g in enumerate(out[1]):
        assert np.array_equal(g, out[0][i % len(one)])
