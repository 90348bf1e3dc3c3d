"""What a plan says of its launch mode: small point masses run whole replans by default and draw nothing ahead; stage by
stage, and for larger ones, each rollout draws the next iteration's tensor paths."""
import pytest

import mtp_workloads as W
import paper_2505_01059_amd as mtp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tensor,gauss,whole", [(256, 32, True), (256, 33, False), (1000, 24, True), (1000, 25, False),
                                                (2000, 20, False)])
def test_draws_ahead_follows_the_mode(tensor, gauss, whole):
    cfg = W.point_mass_config(n_tensor=tensor, n_gauss=gauss, horizon=20, n_elites=16, n_iters=4, n_layers=5, n_width=8)
    plan = mtp.Plan(cfg, device="cuda:0")
    assert plan.draws_ahead() == (not whole)
    plan.set_stage_timing(True)
    assert plan.draws_ahead()
    plan.set_stage_timing(False)
    plan.set_graph_mode(False)
    assert plan.draws_ahead()
    plan.close()
