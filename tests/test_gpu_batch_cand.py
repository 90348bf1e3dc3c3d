"""Candidate tiles of the batched launch against the single plan's, bit for bit.

The batched tile draws all joints of 256 candidates at once (indices packed, graph columns of several joints,
two joints per spline pass); the single plan draws one joint per workgroup.  Same words, same arithmetic: every
cost, elite and moment has to be equal.  Sizes are the tile's edges: horizons under a group of four steps, across
64-step blocks and across the staged chunk of 256; an odd number of joints; more graph columns than fit at once;
every spline form; local samples and tensor paths in one wave.
"""
import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu

BSPLINE, AKIMA, LINEAR = 0, 1, 2

# (links or 0 for the point mass, tensor, local, horizon, layers, width, interp, degree, without replacement)
CASES = [
    (0, 300, 41, 3, 4, 8, BSPLINE, 3, 0),
    (0, 511, 1, 65, 5, 30, AKIMA, 3, 0),
    (0, 100, 300, 257, 6, 19, LINEAR, 3, 0),
    (2, 200, 57, 67, 3, 7, BSPLINE, 2, 0),
    (3, 255, 257, 33, 4, 9, BSPLINE, 1, 0),
    (3, 257, 64, 32, 6, 255, BSPLINE, 5, 0),
    (4, 700, 100, 21, 16, 256, BSPLINE, 4, 0),     # two columns of four at a time
    (7, 513, 65, 127, 12, 62, AKIMA, 3, 0),
    (7, 400, 50, 300, 12, 256, BSPLINE, 3, 0),     # two columns of seven, two chunks
    (7, 300, 40, 18, 5, 11, BSPLINE, 3, 1),
    (12, 130, 20, 260, 9, 33, AKIMA, 3, 1),        # two chunks, columns kept
    (24, 260, 30, 16, 12, 64, BSPLINE, 3, 0),      # ten columns of twenty-four
]


@pytest.mark.parametrize("links,tensor,local,T,layers,width,interp,degree,wor", CASES)
def test_batch_candidates_equal_plan(links, tensor, local, T, layers, width, interp, degree, wor):
    kw = dict(n_tensor=tensor, n_gauss=local, horizon=T, n_layers=layers, n_width=width, interp=interp,
              bspline_degree=degree, n_elites=16, n_iters=3, seed=31 + T)
    cfg = (W.chain_config(n_links=links, **kw) if links else W.point_mass_config(**kw)).replace(sample_wor=wor)
    x0 = W.initial_state(cfg, 5)
    for split in (0, 100):   # whole tiles; one joint of a tile per item
        plan = mtp.Plan(cfg, device="cuda:0")
        plan.set_stage_timing(True)   # stage by stage: the single plan's candidate kernel every iteration
        bt = mtp.Batch([cfg], device="cuda:0")
        bt.set_schedule(split_pct=split)
        for _ in range(2):
            plan.replan(torch.tensor(x0, device="cuda:0"), shift=1)
            bt.replan(bt.pack_x0([x0]), shift=1)
        a, b = plan.buffers(), bt.buffers(0)
        for key in ("cost", "elite_idx", "mu", "sigma"):
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), (key, split)
        bt.close()
        plan.close()
