"""The FP64 update's split over workgroups of 32, 64 or 256 samples: at the sizes where the
split changes, against the weighted sum of the rollout's own effective noise."""
import numpy as np
import pytest
import torch

from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ks,T", [((1,), 1), ((31, 32, 33), 3), ((64, 5, 63), 20), ((2048,), 7), ((2049,), 7),
                                  ((8192,), 4), ((8193,), 4), ((256,) * 8, 100), ((257, 1) * 4, 300)])
def test_split_update_is_the_weighted_noise_sum(Ks, T):
    M, C = params(torch.float64)
    tr = W.spline_track(1)
    probs = [W.Problem(K, T, tr, W.start_state(tr, vx=3.0), W.test_sequences(1, T, seed=b, scale=0.5)[0], b, b)
             for b, K in enumerate(Ks)]
    db = core.DeviceBatch(prep(probs, torch.float64), dtype=torch.float64)
    S, eps = core.rollout(ctx(), db, M, C, 11, want_eps=True)
    w = torch.rand(db.sum_K, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    w[::3] = 0.0
    got = db.controls(core.update(ctx(), db, M, C, 11, w))
    assert ctx().device_errors() == 0
    e, w, o = eps.cpu().numpy(), w.cpu().numpy(), 0
    for b, K in enumerate(Ks):
        ref = np.asarray(probs[b].V, dtype=np.float64) + np.einsum("m,mtd->td", w[o:o + K], e[o:o + K, :T])
        # sums of K terms |w eps| < 0.5 * 3: rounding K * 1.5 * 2^-52, and the clip's cancellation
        assert np.abs(got[b] - ref).max() <= 1e-12 * max(1, K), (b, np.abs(got[b] - ref).max())
        o += K
