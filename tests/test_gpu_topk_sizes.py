"""Elites of small batches on each side of the choice between the selections (one wave, counting, radix), by launch and
fused with the refit: the stable order of the costs, exactly."""
import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("total,elites", [(1, 1), (63, 63), (93, 23), (93, 24), (128, 64), (255, 100), (256, 64), (256, 65),
                                          (256, 256), (257, 64), (257, 65), (257, 257), (260, 65)])
@pytest.mark.parametrize("n_iters", [1, 2])
def test_elites_are_the_stable_order(total, elites, n_iters):
    cfg = W.chain_config(n_links=3, n_tensor=total - (total + 1) // 2, n_gauss=(total + 1) // 2, horizon=9, n_layers=5,
                         n_width=2, n_elites=elites, n_iters=n_iters, interp=W.AKIMA, seed=total + elites)
    x0 = W.initial_state(cfg, 1)
    for graph in (True, False):
        plan = mtp.Plan(cfg, device="cuda:0", use_graph=graph)
        plan.set_stage_timing(not graph)   # selection and refit in launches of their own
        plan.replan(x0, shift=0)
        torch.cuda.synchronize()
        b = plan.buffers()
        cost = b["cost"].cpu().numpy()
        want = np.argsort(cost, kind="stable")[:elites]
        assert np.array_equal(b["elite_idx"].cpu().numpy(), want)
        assert np.array_equal(b["elite_cost"].cpu().numpy(), cost[want])
        plan.close()
