"""The step-pipelined rollouts of small batches give the bits of the one-wave rollout:
a few samples against the first samples of a problem large enough for the latter
(same seed, problem id and iteration, so the same noise), and against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep, rel_err

pytestmark = pytest.mark.gpu


def _problem(K, T, kind, window, seed):
    tr = W.circle_track() if kind == "circle" else W.spline_track(seed)
    tr.window = window
    x0 = W.start_state(tr, 0 if kind == "circle" else 17 * seed % 512, 3.0)
    return W.Problem(K=K, T=T, track=tr, x0=x0, V=W.test_sequences(1, T, seed=seed, scale=0.4)[0], it=seed)


# horizons around the passes (2 and 8 steps) and the rings (8 and 16 slots); sample
# counts around the tiles of 16 and 64, the last of them past the 16-sample rule
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("kind,window", [("spline", 4), ("spline", 2), ("spline", 9), ("circle", 4)])
def test_pipelined_rollout_is_bit_identical(kind, window, dtype):
    M, C = params(dtype)
    for T, Ks in ((1, (1, 16)), (2, (17,)), (8, (63,)), (9, (65,)), (17, (200, 16384)), (33, (1000, 20001))):
        big = prep([_problem(131072, T, kind, window, T)], dtype)[0]
        S, eps = core.rollout(ctx(), core.DeviceBatch([big], dtype=dtype), M, C, 5, want_eps=True)
        for K in Ks:
            p = prep([_problem(K, T, kind, window, T)], dtype)[0]
            s, e = core.rollout(ctx(), core.DeviceBatch([p], dtype=dtype), M, C, 5, want_eps=True)
            assert torch.equal(s, S[:K]) and torch.equal(e, eps[:K]), (T, K)
        n = min(Ks)
        ref, _, margin = oracle.rollout(M, C, big.track, big.x0, big.V, n, 5, 0, big.it)
        ok = margin > 1e-3
        assert rel_err(S[:n].cpu().numpy(), ref)[ok].max(initial=0.0) <= (1e-4 if dtype == torch.float32 else 1e-9)
    assert ctx().device_errors() == 0


def test_pipelined_rollout_nominal_and_ragged():
    M, C = params(torch.float32)
    probs = prep([_problem(K, T, "spline", 4, 3 + i) for i, (K, T) in enumerate(((5, 12), (0, 3), (130, 1), (64, 40)))],
                 torch.float32)
    db = core.DeviceBatch(probs)
    for nominal in (False, True):
        S = core.rollout(ctx(), db, M, C, 9, nominal=nominal)
        o = 0
        for b, p in enumerate(probs):
            if p.K:
                ref, _, margin = oracle.rollout(M, C, p.track, p.x0, p.V, p.K, 9, b, p.it, nominal=nominal)
                ok = margin > 1e-3
                assert rel_err(S[o:o + p.K].cpu().numpy(), ref)[ok].max(initial=0.0) <= 1e-4
            o += p.K
    assert ctx().device_errors() == 0
