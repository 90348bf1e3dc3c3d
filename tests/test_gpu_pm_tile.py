"""The point-mass rollout of a single plan (tiles of 16 candidates, integrated
first, cost terms in parallel) against the batched launch's one-lane rollout:
the same costs and recorded states bit for bit."""
import numpy as np
import pytest

import mtp_workloads as W

pytestmark = pytest.mark.gpu


def _pm(B, T, obs=20, dbg=0):
    return dbg, W.point_mass_config(name=f"B{B}_T{T}_o{obs}_d{dbg}", n_tensor=B - B // 3, n_gauss=B // 3, horizon=T,
                                    n_elites=2, n_iters=2, n_layers=5, n_width=7, n_obstacles=obs, seed=B + T)


CASES = [
    _pm(3, 1), _pm(15, 63), _pm(16, 64), _pm(17, 65), _pm(33, 129, dbg=33), _pm(500, 50, dbg=17), _pm(100, 40, obs=0),
    _pm(100, 40, obs=4), _pm(100, 40, obs=9), _pm(100, 40, obs=40), _pm(60, 30, obs=256),
    # tiles on every compute unit beside the generators, and more tiles than units
    _pm(3584, 20), _pm(3600, 20), _pm(9001, 17),
]


@pytest.mark.parametrize("dbg,cfg", CASES, ids=lambda v: getattr(v, "name", ""))
def test_tile_equals_one_lane(dbg, cfg):
    import torch
    import paper_2505_01059_amd as mtp
    x0 = W.initial_state(cfg, seed=4)
    print(f"[pm tile] {cfg.name}", flush=True)
    plan = mtp.Plan(cfg, device="cuda:0", n_debug_states=dbg)
    plan.replan(x0, shift=0, replan_idx=0)
    bt = mtp.Batch([cfg], device="cuda:0", n_debug_states=[dbg])
    bt.replan(bt.pack_x0([x0]))
    bt.actions()
    torch.cuda.synchronize()
    a, b = plan.buffers(), bt.buffers(0)
    for key in ("cost", "mu", "sigma") + (("X",) if dbg else ()):
        assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), key
    plan.close()
    bt.close()
