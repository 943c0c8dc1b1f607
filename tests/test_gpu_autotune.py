"""The autotuner times what a plan picks by itself, which alone runs its rollouts in a
launch of their own, and drops cache entries from before it did."""
import pytest
import torch

from paper_2302_11719_amd import autotune, core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep

pytestmark = pytest.mark.gpu
AUTO = dict(pipeline=0, block=0, tile=0, grid=0)


@pytest.mark.parametrize("K,T,n_obs", [(33000, 40, 0), (4096, 20, 64)])  # both split plans
def test_tuning_covers_the_automatic_configuration(K, T, n_obs, tmp_path):
    M, C = params(torch.float32)
    p = W.config4(K=K, T=T, n_obs=n_obs) if n_obs else W.config1(K=K, T=T)
    db = core.DeviceBatch(prep([p], torch.float32))
    cache = tmp_path / "tune.txt"
    key = autotune.shape_key(db, torch.cuda.get_device_properties(0).multi_processor_count)
    cache.write_text(f"{key} -1 64 64 0 0.001\n")  # as written before
    r = autotune.tune(ctx(), db, M, C, 3, W.LAMBDA, reps=3, warmup=1, cache=str(cache))
    assert not r.cached
    rows = [row for row in r.table if all(row[k] == v for k, v in AUTO.items())]
    assert len(rows) == 1 and rows[0]["kernel_ms"] > 0
    assert len(r.table) == 1 + len(autotune.candidates(1))
    assert r.best_ms <= rows[0]["kernel_ms"]
    again = autotune.tune(ctx(), db, M, C, 3, W.LAMBDA, cache=str(cache))
    assert again.cached and again.best == r.best
    tuned = autotune.tuned_plan(ctx(), db, M, C, 3, W.LAMBDA, cache=str(cache))
    own = core.Plan(ctx(), db, M, C, 3, W.LAMBDA, **r.best)
    tuned.launch()
    own.launch()
    torch.cuda.synchronize()
    assert torch.equal(tuned.S, own.S) and ctx().device_errors() == 0
    print(r.table[:3], rows, flush=True)


def test_all_zero_candidate_is_the_automatic_configuration():
    """Given by the caller, it is timed as the plan builds it: the two kernels of the split."""
    M, C = params(torch.float32)
    db = core.DeviceBatch(prep([W.config4(K=65536, T=100, n_obs=64)], torch.float32))
    one = dict(pipeline=-1, block=256, tile=256, grid=0)
    r = autotune.tune(ctx(), db, M, C, 3, W.LAMBDA, cands=[one, AUTO], reps=5, warmup=2, cache=None)
    print(r.table, flush=True)
    # (0.10 ms against 0.13 with one launch)
    assert r.best == AUTO and len(r.table) == 2
