"""Weights of more problems than compute units (256 threads per problem, the longer ones in
tiles) against the same problems in small calls."""
import numpy as np
import pytest
import torch

from paper_2302_11719_amd import core

from gpu_helpers import ctx
from test_gpu_weights import _batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("B,largest", [(257, 1025), (257, 8192), (300, 8193), (1025, 20000), (1024, 9000)])
def test_many_problems_have_the_weights_of_small_calls(B, largest, dtype):
    rng = np.random.default_rng(B + largest)
    Ks = [int(k) for k in rng.integers(0, 400, B)]
    Ks[B // 2], Ks[3], Ks[B - 1] = largest, 1024, 2100
    db = _batch(Ks, dtype)
    S = torch.as_tensor(100.0 + 30.0 * rng.random(db.sum_K), dtype=dtype, device="cuda")
    S[torch.as_tensor(rng.random(db.sum_K) < 0.05, device="cuda")] = float("nan")
    w, stats = core.weights(ctx(), db, S, 2.0)
    off = np.concatenate([[0], np.cumsum(Ks)])
    for b in (0, 3, B // 2, B - 1):
        s = S[off[b]:off[b + 1]]
        if not len(s):
            continue
        w1, st1 = core.weights(ctx(), _batch([Ks[b]], dtype), s.clone(), 2.0)
        # the same exponentials, summed in another order: a few units per level of the sums
        tol = 64 * torch.finfo(dtype).eps
        assert torch.allclose(w[off[b]:off[b + 1]], w1, rtol=tol, atol=0)
        assert torch.allclose(stats[b], st1[0], rtol=tol, atol=tol)
    assert ctx().device_errors() == 0
