"""One-problem plans keep the offsets they read at creation (smppi_plan_create), also where
the rollouts run in a launch of their own."""
import pytest
import torch

from paper_2302_11719_amd import core
from paper_2302_11719_amd import workloads as W

from gpu_helpers import ctx, params, prep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,T,n_obs", [(33000, 40, 0), (4096, 20, 64), (2000, 10, 0)])  # two split plans, latency mode
def test_later_offset_changes_are_not_seen(K, T, n_obs):
    M, C = params(torch.float32)
    p = prep([W.config4(K=K, T=T, n_obs=n_obs) if n_obs else W.config1(K=K, T=T)], torch.float32)[0]
    db = core.DeviceBatch([p])
    plan = core.Plan(ctx(), db, M, C, 7, W.LAMBDA)
    plan.launch()
    torch.cuda.synchronize()
    want = [t.clone() for t in (plan.S, plan.V_plus, plan.stats)]
    for t in (plan.S, plan.V_plus, plan.stats):
        t.fill_(float("nan"))
    db.k_off[1] = K // 2  # (smaller: in range of every array)
    db.t_off[1] = T // 2
    db.poly_off[1] = db.poly_off[1] // 2
    plan.launch()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, (plan.S, plan.V_plus, plan.stats)))
    assert ctx().device_errors() == 0
