"""Single plans against the batched launch's narrow rollout forms (a schedule that never splits takes no wide form), bit
for bit: the time-sliced rollout just above one wave group per SIMD and between one and two, over several replans, and
the plans that draw ahead."""
import dataclasses

import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp
from test_gpu_batch import overlap_mix

pytestmark = pytest.mark.gpu


def _sliced(links, contact, uneven, total, T):
    kw = dict(n_links=links, n_tensor=total - 200, n_gauss=200, horizon=T, n_layers=6, n_width=9, n_elites=64, n_iters=2,
              seed=T + links)
    cfg = W.chain_contact_config(ground_y=-2.0, **kw) if contact else W.chain_config(interp=W.AKIMA, **kw)
    if uneven:
        rng = np.random.default_rng(links)
        cfg = cfg.replace(task=dataclasses.replace(cfg.task, lengths=rng.uniform(0.7, 1.3, links).astype(np.float32)))
    return cfg.replace(name=f"sliced{links}_{'contact' if contact else 'plain'}_{'uneven' if uneven else 'even'}_{total}")


CASES = [_sliced(12, False, False, 32800, 16), _sliced(12, False, True, 40000, 19), _sliced(24, False, False, 33300, 17),
         _sliced(24, True, False, 40200, 16), _sliced(24, True, True, 33000, 23)] + overlap_mix()


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_plan_equals_narrow_batch(cfg):
    x0 = W.initial_state(cfg, 2)
    plan, bt = mtp.Plan(cfg, device="cuda:0"), mtp.Batch([cfg], device="cuda:0")
    bt.set_schedule(split_pct=0)
    for _ in range(3):
        plan.replan(torch.tensor(x0, device="cuda:0"), shift=1)
        bt.replan(bt.pack_x0([x0]), shift=1)
        torch.cuda.synchronize()
        assert plan.flags() & 6 == 0
        a, b = plan.buffers(), bt.buffers(0)
        for key in ("cost", "elite_idx", "mu", "sigma"):
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), key
    bt.close()
    plan.close()
