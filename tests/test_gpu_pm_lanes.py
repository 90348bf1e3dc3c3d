"""Point-mass rollouts on both sides of the choice between tiles and eight lanes per candidate, bit for bit those of the
batched launch's one-lane form: the limits in horizon, obstacles and candidates, one obstacle more than the lanes' registers
hold, and the horizons that a tile's threads share out differently."""
import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("total,horizon,obstacles,debug", [
    (16384, 20, 30, 0), (16385, 20, 30, 0), (16385, 20, 33, 0), (16385, 64, 8, 40), (16385, 96, 7, 0), (16385, 63, 0, 3),
    (28672, 64, 20, 0), (28673, 64, 20, 0), (28673, 63, 32, 0), (40001, 17, 25, 7), (17000, 7, 9, 0),
    # one, two and four points of a chunk per thread of a tile
    (900, 16, 20, 0), (900, 17, 30, 5), (900, 32, 20, 0), (900, 33, 9, 0), (900, 65, 20, 900), (8212, 1, 32, 0),
])
def test_point_mass_rollout_equals_batched(total, horizon, obstacles, debug):
    cfg = W.point_mass_config(n_obstacles=obstacles, n_tensor=total - total // 9, n_gauss=total // 9, horizon=horizon,
                              n_layers=6, n_width=9, n_elites=70, n_iters=2, interp=W.AKIMA, seed=total)
    x0 = W.initial_state(cfg, 4)
    plan = mtp.Plan(cfg, device="cuda:0", n_debug_states=debug)
    bt = mtp.Batch([cfg], device="cuda:0", n_debug_states=[debug])
    bt.set_schedule(split_pct=0)
    for _ in range(2):
        plan.replan(x0, shift=1)
        bt.replan(bt.pack_x0([x0]), shift=1)
    torch.cuda.synchronize()
    a, b = plan.buffers(), bt.buffers(0)
    for key in ("cost", "elite_idx", "mu", "sigma") + (("X",) if debug else ()):
        assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), key
    plan.close()
    bt.close()
