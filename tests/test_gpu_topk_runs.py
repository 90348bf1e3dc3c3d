"""Top-E of elite sets ordered by runs of 64: sizes around whole runs and around the two lines of the rule,
batches whose cost images fit in LDS and not, ties and equal costs."""
import numpy as np
import pytest

import mtp_workloads as W
from oracle import planner as OP

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["spread", "ties", "equal"])
@pytest.mark.parametrize("B,E", [(300, 256), (300, 257), (320, 320), (600, 511), (5000, 512), (5000, 513), (16385, 575),
                                 (20011, 831), (1200, 1023), (9000, 1024), (9000, 1025)])
def test_topk_runs(B, E, kind):
    import torch
    import paper_2505_01059_amd as mtp
    cfg = W.point_mass_config(n_tensor=B - 1, n_gauss=1, n_elites=E, n_iters=1)
    plan = mtp.Plan(cfg, device="cuda:0")
    b = plan.buffers()
    rng = np.random.default_rng(B * 7 + E)
    cost = rng.normal(size=B).astype(np.float32)
    if kind == "ties":
        cost = np.round(cost, 2)
    elif kind == "equal":
        cost[:] = np.float32(-1.5)
    print(f"[topk] B={B} E={E} {kind}", flush=True)
    b["cost"].copy_(torch.from_numpy(cost))
    plan.run_stage(mtp.STAGE_TOPK, 0, 0)
    torch.cuda.synchronize()
    assert np.array_equal(b["elite_idx"].cpu().numpy(), OP.top_elites(cost, E))
    plan.close()


@pytest.mark.parametrize("E", [257, 700, 1024])
def test_topk_runs_batch(E):
    import torch
    import paper_2505_01059_amd as mtp
    cfg = W.chain_config(n_links=2, n_tensor=1900, n_gauss=150, horizon=16, n_elites=E, n_iters=2, seed=E)
    x0 = W.initial_state(cfg, 1)
    bt = mtp.Batch([cfg], device="cuda:0")
    bt.replan(bt.pack_x0([x0]), shift=1)
    b = bt.buffers(0)
    torch.cuda.synchronize()
    cost = b["cost"].cpu().numpy()
    assert np.array_equal(b["elite_idx"].cpu().numpy(), OP.top_elites(cost, E))
    bt.close()
