"""Chains in contact inside the batched launch: the narrow rollout form keeps its state in registers.

Spilled to scratch memory, the 24-link form took up to seven times as long as the wide forms, which issue more
instructions for the same candidates; held in registers the two lie within a factor of two of each other.  Times are
compared with each other in one run, the shortest of several replans each.
"""
import dataclasses
import time

import numpy as np
import pytest
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu


def _replan_ms(cfg, split_pct):
    x0 = W.initial_state(cfg, 3)
    bt = mtp.Batch([cfg], device="cuda:0")
    bt.set_schedule(split_pct=split_pct)
    xp = bt.pack_x0([x0])
    best = float("inf")
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        bt.replan(xp, shift=0)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) * 1e3)
    out = {k: bt.buffers(0)[k].cpu().numpy() for k in ("cost", "mu", "sigma")}
    bt.close()
    return best, out


@pytest.mark.parametrize("links,tensor,uneven", [(24, 30000, False), (24, 30000, True), (7, 60000, False)])
def test_narrow_contact_form_stays_in_registers(links, tensor, uneven):
    cfg = W.chain_contact_config(n_links=links, n_tensor=tensor, n_gauss=500, horizon=48, n_layers=6, n_width=9,
                                 n_elites=64, n_iters=2, seed=links, ground_y=-0.5)
    if uneven:
        lengths = np.linspace(0.8, 1.2, links).astype(np.float32)
        cfg = cfg.replace(task=dataclasses.replace(cfg.task, lengths=lengths))
    narrow, a = _replan_ms(cfg, 0)
    chosen, b = _replan_ms(cfg, 100)
    print(f"[contact] {links} links: narrow {narrow:.2f} ms, chosen {chosen:.2f} ms", flush=True)
    for key in a:
        assert np.array_equal(a[key], b[key]), key
    assert narrow < 2.0 * chosen
