"""FP32 rollouts with obstacles as a pipeline of waves: few samples give the bits of the
one-wave rollout (the first samples of a problem too large for the pipeline), and the
oracle's costs."""
import pytest
import torch

from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import band_mask, ctx, oracle_iteration, params, prep, rel_err

pytestmark = pytest.mark.gpu
BAND = 1e-3


def _problem(K, T, n_obs, window=4, circle=False):
    p = W.config4(K=K, T=T, n_obs=n_obs)
    if circle:  # the same obstacles beside a circular centre line
        c = W.circle_track(10.0, 1.0)
        c.obs, p.track, p.x0 = p.track.obs, c, W.start_state(c, vx=3.0)
    p.track.window = window
    p.V = W.test_sequences(1, T, seed=T, scale=0.5)[0]
    return p


@pytest.mark.parametrize("T,n_obs,window,circle", [(1, 64, 4, False), (2, 1, 4, False), (3, 17, 2, False),
                                                   (8, 64, 4, False), (9, 5, 9, False), (33, 40, 4, False),
                                                   (10, 3, 4, True)])
def test_pipelined_obstacle_rollout_is_bit_identical(T, n_obs, window, circle):
    M, C = params(torch.float32)

    def run(K):
        db = core.DeviceBatch(prep([_problem(K, T, n_obs, window, circle)], torch.float32), dtype=torch.float32)
        return core.rollout(ctx(), db, M, C, 5, want_eps=True)

    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    S, eps = run(7 * 64 * n_cu)
    for K in (1, 63, 64, 65, 1000):
        s, e = run(K)
        assert torch.equal(s, S[:K]) and torch.equal(e, eps[:K])
    assert ctx().device_errors() == 0


def test_pipelined_obstacle_batch_vs_oracle():
    """Ragged problems: the tolerance and the band of the ragged parity test."""
    probs = prep([_problem(K, T, n) for K, T, n in ((70, 12, 3), (1, 1, 64), (130, 25, 16))], torch.float32)
    for b, p in enumerate(probs):
        p.pid = b  # the noise's problem index is the position in the batch
    M, C = params(torch.float32)
    db = core.DeviceBatch(probs, dtype=torch.float32)
    S = db.per_problem(core.rollout(ctx(), db, M, C, 9))
    for b, p in enumerate(probs):
        r = oracle_iteration(p, M, C, 9, W.LAMBDA)
        ok = band_mask(r["margin"], BAND, f"problem {b}", S[b], r["S"], 1e-4)
        assert rel_err(S[b], r["S"])[ok].max() <= 1e-4
