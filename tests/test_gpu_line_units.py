"""Chains of two and three links on both sides of the choice between the two units their rollout is compiled in: with
the generator beside it and alone, the values are the batched launch's bit for bit."""
import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links,total,horizon,wor", [
    (2, 900, 16, 0), (2, 8192, 20, 1), (2, 8193, 20, 1), (3, 900, 95, 0), (3, 900, 96, 0), (3, 9001, 17, 1),
])
def test_rollout_equals_batched(links, total, horizon, wor):
    # without replacement nothing is drawn ahead: the rollout is alone in its launch
    cfg = W.chain_config(n_links=links, n_tensor=total - total // 9, n_gauss=total // 9, horizon=horizon, n_layers=6,
                         n_width=9, n_elites=40, n_iters=2, interp=W.AKIMA, seed=total).replace(sample_wor=wor)
    x0 = W.initial_state(cfg, 4)
    plan, bt = mtp.Plan(cfg, device="cuda:0"), mtp.Batch([cfg], device="cuda:0")
    assert plan.draws_ahead() == (wor == 0)
    bt.set_schedule(split_pct=0)
    for _ in range(2):
        plan.replan(x0, shift=1)
        bt.replan(bt.pack_x0([x0]), shift=1)
    torch.cuda.synchronize()
    a, b = plan.buffers(), bt.buffers(0)
    for key in ("cost", "elite_idx", "mu", "sigma"):
        assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), key
    plan.run_stage(mtp.STAGE_ROLLOUT, 1, 0)   # alone, on the controls as they stand
    torch.cuda.synchronize()
    assert np.array_equal(a["cost"].cpu().numpy(), b["cost"].cpu().numpy())
    plan.close()
    bt.close()
