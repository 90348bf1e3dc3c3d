"""Selection by one wave in the refit's launch against the staged selection, bit for bit: batches and elite sets on
both sides of the rule's lines, fewer candidates than lanes, more tiles than four per compute unit, and costs that
are all equal (and zero)."""
import dataclasses

import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu

# (links or 0 for the point mass, tensor, local, horizon, elites, equal costs, without replacement)
CASES = [
    (3, 500, 61, 32, 16, False, False),
    (4, 20, 4, 3, 24, False, False),      # every candidate an elite, fewer than a wave's lanes
    (2, 700, 324, 9, 64, False, False),   # 1024 candidates
    (2, 701, 324, 9, 64, False, False),   # one more
    (7, 800, 100, 21, 65, False, False),  # one elite more
    (12, 300, 300, 66, 33, False, True),
    (24, 200, 40, 171, 20, False, False),  # 1032 tiles
    (0, 600, 90, 40, 40, False, False),
    (0, 600, 90, 40, 40, True, False),
]


@pytest.mark.parametrize("links,tensor,local,T,elites,equal,wor", CASES)
def test_select_by_wave_equals_staged(links, tensor, local, T, elites, equal, wor):
    kw = dict(n_tensor=tensor, n_gauss=local, horizon=T, n_layers=5, n_width=14, n_elites=elites, n_iters=4, seed=T)
    cfg = (W.chain_config(n_links=links, **kw) if links else W.point_mass_config(**kw)).replace(sample_wor=int(wor))
    if equal:
        cfg = cfg.replace(task=dataclasses.replace(cfg.task, goal_weight=0.0, obstacle_penalty=0.0, ctrl_weight=0.0))
    x0 = torch.tensor(W.initial_state(cfg, 3), device="cuda:0")
    got = []
    for staged in (False, True):
        plan = mtp.Plan(cfg, device="cuda:0")
        plan.set_stage_timing(staged)
        for _ in range(3):
            plan.replan(x0, shift=1)
        torch.cuda.synchronize()
        assert plan.flags() & 6 == 0
        got.append({k: v.cpu().numpy().copy() for k, v in plan.buffers().items()
                    if k in ("cost", "elite_idx", "elite_cost", "weights", "mu", "sigma", "action")})
        plan.close()
    if equal:
        assert np.all(got[0]["cost"] == 0.0)
    for key, a in got[0].items():
        assert np.array_equal(a, got[1][key]), key
