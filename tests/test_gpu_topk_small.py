"""Top-E on batches below and just above the boundary bin's 256 keys: no radix
pass, one pass, and costs that are all equal (the index radix decides)."""
import numpy as np
import pytest

import mtp_workloads as W
from oracle import planner as OP

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["spread", "ties", "equal"])
@pytest.mark.parametrize("B,E", [(2, 1), (2, 2), (65, 64), (256, 255), (257, 1), (257, 257), (700, 300), (1024, 1023)])
def test_topk_small(B, E, kind):
    import torch
    import paper_2505_01059_amd as mtp
    cfg = W.point_mass_config(n_tensor=B - 1, n_gauss=1, n_elites=E, n_iters=1)
    plan = mtp.Plan(cfg, device="cuda:0")
    b = plan.buffers()
    rng = np.random.default_rng(B * 7 + E)
    cost = rng.normal(size=B).astype(np.float32)
    if kind == "ties":
        cost = np.round(cost, 1)
    elif kind == "equal":
        cost[:] = np.float32(3.25)
    print(f"[topk] B={B} E={E} {kind}", flush=True)
    b["cost"].copy_(torch.from_numpy(cost))
    plan.run_stage(mtp.STAGE_TOPK, 0, 0)
    torch.cuda.synchronize()
    assert np.array_equal(b["elite_idx"].cpu().numpy(), OP.top_elites(cost, E))
    plan.close()
