"""Which kernel a call takes does not change what it computes: sizes on both sides of the
pipelines' rules (workgroups per compute unit, their LDS, short horizons) against small
calls, which always run as pipelines."""
import numpy as np
import pytest
import torch

from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep

pytestmark = pytest.mark.gpu
F32, F64 = torch.float32, torch.float64


def _problem(K, T, n_s=512, n_obs=0, b=0):
    tr = W.spline_track(b, n_s=n_s)
    if n_obs:
        tr.obs = W.obstacles(tr, b, n_obs, keep_clear=1.0)
    return W.Problem(K=K, T=T, track=tr, x0=W.start_state(tr), V=W.test_sequences(1, T, seed=b, scale=0.4)[0], pid=0,
                     it=b)


@pytest.mark.parametrize("dtype,n_s,n_obs,K,Ts", [
    (F32, 512, 0, 45000, (4, 5)), (F32, 512, 0, 65536, (11, 12)), (F32, 3000, 0, 8192, (1, 6)),
    (F32, 3000, 8, 30000, (2, 40)), (F32, 1024, 8, 98304, (12, 39, 40)), (F32, 512, 8, 98304, (3, 11, 12)),
    (F64, 512, 0, 30000, (2, 3)), (F64, 1500, 0, 30000, (19, 20))])
def test_rollouts_have_the_bits_of_a_small_call(dtype, n_s, n_obs, K, Ts):
    M, C = params(dtype)
    for T in Ts:
        S = [core.rollout(ctx(), core.DeviceBatch(prep([_problem(k, T, n_s, n_obs)], dtype), dtype=dtype), M, C, 5)
             for k in (200, K)]
        assert torch.equal(S[0], S[1][:200]), T
    assert ctx().device_errors() == 0


@pytest.mark.parametrize("dtype,n,K,Ts", [(F32, 8000, 70000, (3, 4, 5, 6)), (F32, 1024, 90000, (5, 6)),
                                          (F64, 8000, 20000, (4, 5))])
def test_curvilinear_rollouts_have_the_bits_of_a_small_call(dtype, n, K, Ts):
    M, C = params(dtype)
    f = (lambda a: np.asarray(a, np.float32).astype(np.float64)) if dtype == F32 else np.asarray
    for T in Ts:
        S = []
        for k in (200, K):
            p = prep([_problem(k, T)], dtype)[0]
            kappa, ds = W.curvature_table(p.track, n)
            ct = core.CurvTrackArrays([(f(kappa), float(f(ds)))], [p.track.half_width], dtype=dtype)
            x0 = torch.as_tensor(W.start_state_c8(vx=3.0), dtype=dtype, device="cuda")
            S.append(core.rollout_curvilinear(ctx(), core.DeviceBatch([p], dtype=dtype), ct, M,
                                              W.wheels_f32() if dtype == F32 else W.WHEELS, C, 5, x0=x0))
        assert torch.equal(S[0], S[1][:200]), T
    assert ctx().device_errors() == 0


@pytest.mark.parametrize("dtype,B,Ts,tol", [(F32, 520, (1, 2, 3), 2e-6), (F64, 260, (4, 5), 1e-14)])
@pytest.mark.parametrize("curvilinear", [False, True])
def test_adjoints_agree_with_a_problem_alone(dtype, B, Ts, tol, curvilinear):
    """Single samples over at most five steps: some 200 chained operations, whose roundings
    of half a unit (6e-8, 1e-16) and random sign add up to 14 of them, well below tol."""
    M, C = params(dtype)
    wh = W.wheels_f32() if dtype == F32 else W.WHEELS
    for T in Ts:
        probs = prep([_problem(1, T, b=b % 8) for b in range(B)], dtype)
        for b, p in enumerate(probs):
            p.pid = b

        def grad(ps, pid_base):
            db = core.DeviceBatch(ps, dtype=dtype, pid_base=pid_base)
            g = torch.ones(db.sum_K, dtype=dtype, device="cuda")
            if not curvilinear:
                return db.controls(core.rollout_backward(ctx(), db, M, C, 5, g, W.OBJ_TOTAL))
            tabs = [W.curvature_table(p.track, 256) for p in ps]
            ct = core.CurvTrackArrays(tabs, [p.track.half_width for p in ps], dtype=dtype)
            x0 = torch.as_tensor(np.concatenate([W.start_state_c8(vx=3.0) for _ in ps]), dtype=dtype, device="cuda")
            return db.controls(core.rollout_backward_curvilinear(ctx(), db, ct, M, wh, C, 5, g, W.OBJ_TOTAL, x0=x0))

        got = grad(probs, 0)
        for b in (0, 7, B - 1):
            ref = grad([probs[b]], b)[0]
            assert np.abs(got[b] - ref).max() <= tol * np.abs(ref).max(), (T, b)
    assert ctx().device_errors() == 0


@pytest.mark.parametrize("B,T", [(1537, 8), (2048, 5), (2048, 16), (2049, 8)])
def test_fp64_adjoints_in_one_round_agree_with_a_problem_alone(B, T):
    """Both sides of 7 and 8 one-wave workgroups per compute unit.  Single samples over up to
    16 steps: some 700 chained operations, whose roundings of 1e-16 add up to 26 of them."""
    M, C = params(F64)
    probs = prep([_problem(1, T, n_s=32, b=b % 8) for b in range(B)], F64)

    def grad(ps, pid_base):
        db = core.DeviceBatch(ps, dtype=F64, pid_base=pid_base)
        return db.controls(core.rollout_backward(ctx(), db, M, C, 5, torch.ones(db.sum_K, dtype=F64, device="cuda"),
                                                 W.OBJ_TOTAL))

    for b, p in enumerate(probs):
        p.pid = b
    got = grad(probs, 0)
    for b in (0, 7, B - 1):
        ref = grad([probs[b]], b)[0]
        assert np.abs(got[b] - ref).max() <= 3e-14 * np.abs(ref).max(), b
    assert ctx().device_errors() == 0
