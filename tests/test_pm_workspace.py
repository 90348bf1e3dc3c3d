"""A point mass's workspace does not grow with its iterations, but for the cost entropy's one value each (host only)."""
import pytest

import mtp_workloads as W
from paper_2505_01059_amd import _native as N


@pytest.mark.parametrize("tensor,gauss", [(255, 1), (992, 32)])
def test_workspace_is_bounded_in_the_iterations(tensor, gauss):
    def size(n_iters):
        return N.workspace_bytes(W.point_mass_config(n_tensor=tensor, n_gauss=gauss, horizon=20, n_elites=16,
                                                     n_iters=n_iters, n_layers=5, n_width=8))
    assert size(65535) - size(100) <= 4 * 65535 + 256
    assert size(100) - size(10) <= 4 * 1024 * 64 + 1024
