"""A plan's lanes per candidate leave the units that drawing the next tensor paths needs: a plan of fewer candidates,
just below the size up to which a wider rollout form fits, is not slower than one just above it, and the values are
those of the batched launch.

The two sizes do about the same work, so their times lie within a few per cent of each other; with most units given
to the rollout the smaller one took up to 1.9 times as long.
"""
import time

import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu

_COMMON = dict(n_layers=9, n_width=40, n_iters=4, n_elites=128)


def _sizes(total):
    return dict(n_tensor=total - total // 9, n_gauss=total // 9, **_COMMON)


def _chain(links, interp, horizon):
    return lambda total: W.chain_config(n_links=links, interp=interp, horizon=horizon, seed=links, **_sizes(total))


def _contact(links, horizon, replicas):
    return lambda total: W.chain_contact_config(n_links=links, horizon=horizon, n_replicas=replicas, ground_y=-4.0,
                                                seed=links + replicas, **_sizes(total))


def _point_mass(horizon):
    return lambda total: W.point_mass_config(n_obstacles=8, interp=W.LINEAR, horizon=horizon, seed=horizon,
                                             **_sizes(total))


PAIRS = {
    "24 links": (_chain(24, W.BSPLINE, 16), 14000, 14600),
    "12 links": (_chain(12, W.LINEAR, 64), 14000, 14600),
    "4 links": (_chain(4, W.LINEAR, 64), 28000, 29500),
    "24 links in contact": (_contact(24, 16, 1), 14000, 14600),
    "two models": (_contact(24, 16, 2), 14600, 28600),
    "models that share units": (_contact(7, 24, 2), 32700, 45800),
    "7 links": (_chain(7, W.AKIMA, 128), 14000, 14600),
    "point mass": (_point_mass(64), 5000, 7300),
}


def _replan_ms(cfg):
    plan = mtp.Plan(cfg, device="cuda:0")
    x0 = torch.tensor(W.initial_state(cfg, 1), device="cuda:0")
    best = float("inf")
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(4):
            plan.replan(x0, shift=1)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) * 250.0)
    plan.close()
    return best


@pytest.mark.parametrize("name", PAIRS)
def test_fewer_candidates_are_not_slower(name):
    make, below, above = PAIRS[name]
    a, b = _replan_ms(make(below)), _replan_ms(make(above))
    print(f"[lanes] {name}: {below} candidates {a:.3f} ms, {above} {b:.3f} ms", flush=True)
    assert a < 1.25 * b


@pytest.mark.parametrize("name", PAIRS)
def test_values_at_the_limits(name):
    make, below, above = PAIRS[name]
    for total in (below, above):
        cfg = make(total).replace(n_iters=2)
        x0 = W.initial_state(cfg, 2)
        plan, bt = mtp.Plan(cfg, device="cuda:0"), mtp.Batch([cfg], device="cuda:0")
        bt.set_schedule(split_pct=0)
        for _ in range(2):
            plan.replan(x0, shift=1)
            bt.replan(bt.pack_x0([x0]), shift=1)
        torch.cuda.synchronize()
        a, b = plan.buffers(), bt.buffers(0)
        for key in ("cost", "elite_idx", "mu", "sigma"):
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), (total, key)
        plan.close()
        bt.close()
