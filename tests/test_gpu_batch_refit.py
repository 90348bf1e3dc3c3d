"""Refit items of the batched launch (four outputs of a wave at a time) against the single plan's, bit for bit:
elite sets around the lanes of a wave and the registers of the tile, outputs that do not fill the last item."""
import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links,T,E", [(7, 33, 1), (7, 33, 63), (2, 8, 64), (3, 43, 65), (12, 11, 500), (2, 65, 1024),
                                       (2, 65, 1025), (0, 9, 40)])
def test_batch_refit_equals_plan(links, T, E):
    kw = dict(n_tensor=1400, n_gauss=160, horizon=T, n_layers=5, n_width=9, n_elites=E, n_iters=2, seed=E + T)
    cfg = W.chain_config(n_links=links, **kw) if links else W.point_mass_config(**kw)
    x0 = W.initial_state(cfg, 4)
    plan = mtp.Plan(cfg, device="cuda:0")
    plan.replan(torch.tensor(x0, device="cuda:0"), shift=1)
    bt = mtp.Batch([cfg], device="cuda:0")
    for outputs in (16, 64):
        bt.close()
        bt = mtp.Batch([cfg], device="cuda:0")
        bt.set_schedule(split_pct=0, refit_outputs=outputs)
        bt.replan(bt.pack_x0([x0]), shift=1)
        a, b = plan.buffers(), bt.buffers(0)
        for key in ("elite_idx", "mu", "sigma", "action"):
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), (key, outputs)
    bt.close()
    plan.close()
