"""Two steps per launch (march2): runs of steps give the state, the totals and
the fields of one-step launches, bit for bit."""
import os

import numpy as np
import pytest

import paper_2409_16781_amd as lbm
from paper_2409_16781_amd import inputs

from gpu_util import make_lattice, say

pytestmark = pytest.mark.gpu


def _lattice(cfg, two, codec="f32"):
    os.environ["LB_TWO_STEP"] = two
    try:
        return make_lattice(cfg, codec)
    finally:
        os.environ.pop("LB_TWO_STEP", None)


def _cfg(shape, force, seed, flags=None):
    return dict(name="two_step", shape=shape, tau=0.57, force=force, flags=flags,
                rho=1.0 + inputs.uniform_noise(shape, 1e-3, seed), u=inputs.uniform_noise((3,) + shape, 3e-2, seed + 1))


# rows of one and several tiles of 64 columns, the last one of 1, 33 and 64;
# one plane, fewer than a tile, several tiles with a short last one; marches
# of one row and of odd and even numbers of rows (LB_TWO_STEP=2: also where
# two one-step launches are faster)
@pytest.mark.parametrize("force", [(0.0, 0.0, 0.0), (1e-5, -2e-5, 3e-5)])
@pytest.mark.parametrize("shape", [(1, 1, 5), (1, 9, 64), (3, 2, 65), (13, 7, 64), (14, 40, 97), (29, 33, 128),
                                   (16, 64, 192), (40, 100, 33)])
def test_two_step_runs_equal_single_steps(shape, force):
    cfg = _cfg(shape, force, 41)
    a, b = _lattice(cfg, "2"), _lattice(cfg, "0")
    assert a.query(13) == 2 and b.query(13) == 1
    say(f"[gpu] two-step {shape} force={force}")
    for n in (2, 5, 1, 8, 70):
        a.step(n)
        b.step(n)
    assert np.array_equal(a.get_f().view(np.uint32), b.get_f().view(np.uint32))
    assert np.array_equal(a.sums(86).view(np.uint64), b.sums(86).view(np.uint64))
    c = _lattice(cfg, "2")
    assert lbm.lib().lb_step_noalloc(c.handle, 86) == lbm.LB_OK, lbm.last_error()
    assert np.array_equal(c.get_f().view(np.uint32), b.get_f().view(np.uint32))
    assert np.array_equal(c.sums(86).view(np.uint64), b.sums(86).view(np.uint64))
    for n in (4, 3, 1, 67):
        ra, ua = a.step_macros(n)
        rb, ub = b.step_macros(n)
        assert np.array_equal(ra.cpu().numpy(), rb.cpu().numpy()), n
        assert np.array_equal(ua.cpu().numpy(), ub.cpu().numpy()), n
    for lat in (a, b, c):
        lat.close()


@pytest.mark.parametrize("shape", [(3, 2, 65), (14, 40, 97)])
def test_two_step_runs_with_a_force_field_set_and_cleared(shape):
    """A per-site force sends the lattice to one-step launches (of another
    totals format) until it is cleared."""
    import torch

    cfg = _cfg(shape, (1e-5, 2e-5, 0.0), 47)
    fx = torch.from_numpy(inputs.uniform_noise(shape, 1e-4, 48).astype(np.float32)).cuda()
    a, b = _lattice(cfg, "2"), _lattice(cfg, "0")
    for n in (6, 67):
        for lat in (a, b):
            lat.set_force_field(fx)
            lat.step(n)
            lat.set_force_field(None)
            lat.step(n)
    assert np.array_equal(a.get_f().view(np.uint32), b.get_f().view(np.uint32))
    assert np.array_equal(a.sums(146).view(np.uint64), b.sums(146).view(np.uint64))
    a.close()
    b.close()


def test_graph_replays_of_two_step_runs():
    """Captured runs (64 steps and more) replayed several times, of even and
    odd numbers of two-step launches, with eager steps in between."""
    cfg = _cfg((20, 48, 128), (1e-5, 0.0, 0.0), 5)
    a, b = _lattice(cfg, "2"), _lattice(cfg, "0")
    total = 0
    for n in (64, 64, 66, 66, 66, 3, 67, 67, 2100):
        a.step(n)
        a.sync()
        total += n
    for _ in range(total):
        b.step(1)
    assert np.array_equal(a.get_f().view(np.uint32), b.get_f().view(np.uint32))
    assert np.array_equal(a.sums(total).view(np.uint64), b.sums(total).view(np.uint64))
    a.close()
    b.close()
