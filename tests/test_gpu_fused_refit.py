"""Selection and refit in one launch against the two launches, bit for bit.

A replan runs them as one kernel where each refit tile has a compute unit of its own and the costs fit the
selection's LDS; stage timing runs every stage alone.  Sizes lie on both sides of those lines, with next samples
drawn ahead and without, and elite sets from one to more than the refit keeps in registers.
"""
import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu

# (links or 0 for the point mass, tensor, local, horizon, elites, iterations, interp, without replacement)
CASES = [
    (3, 500, 61, 32, 16, 4, 0, 0),
    (3, 60, 4, 2, 1, 3, 1, 0),          # one elite, one tile per joint
    (7, 8192, 1024, 127, 128, 2, 1, 0),
    (4, 1500, 200, 256, 26, 3, 0, 0),   # 256 tiles
    (4, 1500, 200, 257, 26, 3, 0, 0),   # 260 tiles: two launches
    (12, 700, 80, 33, 20, 3, 1, 1),
    (2, 2500, 500, 40, 1100, 3, 0, 0),  # elites re-read by the refit
    (0, 3000, 341, 77, 52, 4, 1, 0),
    (0, 200, 5000, 9, 40, 2, 2, 0),     # more local samples than a workgroup draws at once
    (2, 16000, 384, 20, 64, 3, 1, 0),   # 16384 candidates
    (2, 16000, 385, 20, 64, 3, 1, 0),   # one more: two launches
]


@pytest.mark.parametrize("links,tensor,local,T,elites,iters,interp,wor", CASES)
def test_one_launch_equals_two(links, tensor, local, T, elites, iters, interp, wor):
    kw = dict(n_tensor=tensor, n_gauss=local, horizon=T, n_layers=6, n_width=20, interp=interp, n_elites=elites,
              n_iters=iters, seed=17 + T)
    cfg = (W.chain_config(n_links=links, **kw) if links else W.point_mass_config(**kw)).replace(sample_wor=wor)
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
    assert len(got[0]) >= 5
    for key, a in got[0].items():
        assert np.array_equal(a, got[1][key]), key
