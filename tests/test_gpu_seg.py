"""The time-sliced pair-lane rollout against the batched launch's plain one, bit for bit.

Just above one wave group per SIMD (every hand-over between segments is waited for) and between one and two;
chains of 12 and 24 links, with and without contact, equal and uneven links; several replans, so that graph replays
find the hand-over flags of the launch before.
"""
import dataclasses

import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu


def _config(links, contact, uneven, tensor, local, T):
    kw = dict(n_links=links, n_tensor=tensor, n_gauss=local, horizon=T, n_layers=6, n_width=9, n_elites=64, n_iters=2,
              seed=T + links)
    cfg = W.chain_contact_config(ground_y=-2.0, **kw) if contact else W.chain_config(interp=1, **kw)
    if uneven:
        rng = np.random.default_rng(links)
        cfg = cfg.replace(task=dataclasses.replace(
            cfg.task, lengths=rng.uniform(0.7, 1.3, links).astype(np.float32),
            masses=rng.uniform(0.7, 1.3, links).astype(np.float32)))
    return cfg


@pytest.mark.parametrize("links,contact,uneven,tensor,local,T", [
    (12, False, False, 32700, 100, 16),    # 1025 groups
    (12, False, True, 39000, 1003, 19),
    (24, False, False, 33000, 289, 17),
    (24, True, False, 40100, 77, 16),
    (24, True, True, 33000, 11, 23),
])
def test_time_sliced_equals_plain(links, contact, uneven, tensor, local, T):
    cfg = _config(links, contact, uneven, tensor, local, T)
    x0 = W.initial_state(cfg, 2)
    plan = mtp.Plan(cfg, device="cuda:0")
    bt = mtp.Batch([cfg], device="cuda:0")
    for _ in range(4):
        plan.replan(torch.tensor(x0, device="cuda:0"), shift=1)
        bt.replan(bt.pack_x0([x0]), shift=1)
        torch.cuda.synchronize()
        assert plan.flags() & 6 == 0
        a, b = plan.buffers(), bt.buffers(0)
        for key in ("cost", "elite_idx", "mu", "sigma"):
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), key
    bt.close()
    plan.close()
