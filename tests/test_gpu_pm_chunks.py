"""Long whole point-mass replans run in chunks of 64 iterations: every buffer is the staged kernels' bit for bit with a
chunk exactly filled, begun by one iteration and repeated."""
import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_iters", [63, 64, 65, 129])
@pytest.mark.parametrize("tensor,gauss", [(250, 5), (0, 20)])
def test_chunked_replan_equals_staged(n_iters, tensor, gauss):
    cfg = W.point_mass_config(n_tensor=tensor, n_gauss=gauss, horizon=21, n_elites=16, n_iters=n_iters, n_layers=5,
                              n_width=7, n_obstacles=9, seed=n_iters, smoothing=0.2)
    whole, staged = mtp.Plan(cfg, device="cuda:0"), mtp.Plan(cfg, device="cuda:0", use_graph=False)
    for seed, shift in ((0, 0), (1, 3)):
        x0 = W.initial_state(cfg, seed)
        for p in (whole, staged):
            p.replan(x0, shift=shift)
        torch.cuda.synchronize()
        a, b = whole.buffers(), staged.buffers()
        assert whole.flags() == staged.flags()
        for key in ("U", "cost", "elite_idx", "elite_cost", "weights", "mu", "sigma", "x0", "action"):
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), (key, shift)
    whole.close()
    staged.close()
