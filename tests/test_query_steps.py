"""lb_query(13) is the number of steps that one launch of a run takes now."""
import pytest
import torch

import paper_2409_16781_amd as lbm

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def test_steps_of_a_launch_follow_the_force_field():
    require_gpu()
    lat = lbm.Lattice(64, 64, 64, 0.7)
    assert lat.query(13) == 2
    lat.set_force_field(torch.zeros((64, 64, 64), dtype=torch.float32, device="cuda"))
    assert lat.query(13) == 1
    lat.set_force_field(None)
    assert lat.query(13) == 2
    lat.close()
