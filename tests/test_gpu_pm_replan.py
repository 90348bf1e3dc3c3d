"""Whole point-mass replans: a plan's replan runs in two kernels (all
iterations' tensor paths at once, then the iterations), the launch-by-launch
mode runs the staged kernels.  Both do the same operations in the same order:
every buffer a caller can look at agrees bit for bit."""
import numpy as np
import pytest

import mtp_workloads as W

pytestmark = pytest.mark.gpu


def _pm(P, G, T, E, K=3, L=5, Wd=7, interp=W.BSPLINE, p=3, obs=20, **k):
    return W.point_mass_config(name=f"P{P}_G{G}_T{T}_E{E}_K{K}_L{L}x{Wd}_i{interp}p{p}_o{obs}", n_tensor=P, n_gauss=G,
                               horizon=T, n_elites=E, n_iters=K, n_layers=L, n_width=Wd, interp=interp,
                               bspline_degree=p, n_obstacles=obs, seed=P + T, **k)


CASES = [
    _pm(255, 1, 20, 16, K=10, Wd=30),                       # the nominal alone beside tensor paths
    _pm(250, 4, 20, 16), _pm(250, 5, 20, 16), _pm(250, 16, 20, 16), _pm(250, 17, 20, 16),   # tile widths
    _pm(256, 32, 50, 16, K=10, L=4, Wd=8),                  # a full tile of local candidates
    _pm(0, 30, 37, 30, K=3), _pm(1, 1, 1, 1, K=1), _pm(1, 2, 3, 3, K=2), _pm(40, 23, 9, 63), _pm(40, 24, 9, 64),
    _pm(100, 17, 64, 63, interp=W.AKIMA, L=2), _pm(100, 17, 65, 64, interp=W.AKIMA, L=3),
    _pm(90, 16, 129, 20, interp=W.AKIMA, L=4), _pm(290, 26, 77, 20, interp=W.AKIMA, L=6, Wd=19),
    _pm(400, 9, 128, 33, interp=W.LINEAR), _pm(400, 20, 63, 31, p=2), _pm(300, 20, 33, 30, p=5, L=9),
    _pm(700, 10, 45, 30, obs=0), _pm(700, 10, 45, 30, obs=9), _pm(700, 10, 45, 30, obs=40), _pm(70, 30, 45, 30, obs=256),
    _pm(1011, 13, 256, 18, K=2, L=16, Wd=64),               # the largest of every size held on chip
    _pm(992, 32, 103, 44, K=2, smoothing=0.3),
    _pm(300, 30, 50, 20, temperature=np.float32(np.inf)),
    # few distinct paths: many equal costs, more of them at the boundary than the short list holds
    _pm(600, 8, 12, 40, L=4, Wd=1), _pm(600, 8, 12, 40, L=4, Wd=2), _pm(900, 1, 12, 64, L=4, Wd=1, K=1),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_whole_replan_equals_staged(cfg):
    import torch
    import paper_2505_01059_amd as mtp
    print(f"[pm] {cfg.name}", flush=True)
    whole = mtp.Plan(cfg, device="cuda:0")
    staged = mtp.Plan(cfg, device="cuda:0", use_graph=False)
    x0 = [W.initial_state(cfg, seed=s) for s in range(3)]
    for x, shift in zip(x0, (0, 1, cfg.horizon + 2)):
        for p in (whole, staged):
            p.replan(x, shift=shift)
        torch.cuda.synchronize()
        a, b = whole.buffers(), staged.buffers()
        assert whole.flags() == staged.flags()
        for key in ("Z", "I", "U", "cost", "elite_idx", "elite_cost", "weights", "mu", "sigma", "x0", "action"):
            if cfg.n_tensor == 0 and key in ("Z", "I"):
                continue
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), (key, shift)
    # modes may alternate from one replan to the next
    for p in (whole, staged):
        p.set_graph_mode(p is staged)
        p.replan(x0[0], shift=2)
    torch.cuda.synchronize()
    assert np.array_equal(whole.buffers()["mu"].cpu().numpy(), staged.buffers()["mu"].cpu().numpy())
    whole.close()
    staged.close()
