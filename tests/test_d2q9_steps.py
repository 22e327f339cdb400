"""Several D2Q9 steps per launch (march2d): runs of steps give the state and
the totals of one-step launches, bit for bit."""
import os

import numpy as np
import pytest
import torch

import paper_2409_16781_amd as lbm
from paper_2409_16781_amd import inputs

from gpu_util import say

pytestmark = pytest.mark.gpu


def _flags(kind, nx, ny):
    if kind == "box":
        return None
    if kind == "cavity" and nx > 2 and ny > 2:
        return inputs.cavity_flags(nx, ny)
    rng = np.random.default_rng(5)
    return rng.choice(np.array([0, 1, 2], np.uint8), size=(ny, nx), p=[0.8, 0.15, 0.05])


def _lattice(nx, ny, flags, most, variant):
    env = {"LB_STEPS2D": str(most), "LB_KERNEL2D": str(variant)}
    os.environ.update(env)
    try:
        lat = lbm.Lattice2D(nx, ny, 0.58, flags=flags, lid=(0.05, -0.02))
    finally:
        for k in env:
            os.environ.pop(k, None)
    lat.init_eq(torch.from_numpy(1.0 + inputs.uniform_noise((ny, nx), 1e-3, 3)).cuda(),
                torch.from_numpy(inputs.uniform_noise((2, ny, nx), 3e-2, 4)).cuda())
    return lat


def _sums(lat, k):
    """The last k totals' bits, or the error of a run that blew up."""
    try:
        return lat.sums(k).tobytes()
    except lbm.LBError as e:
        return str(e)


# one strip of columns and several, with a short last one of 1 vector and
# more; odd lengths of row; chunks of one row, fewer rows than the halo,
# several chunks with a short last one; scattered walls and lid sites on every
# strip edge
@pytest.mark.parametrize("kind", ["box", "cavity", "scattered"])
@pytest.mark.parametrize("nx,ny,variant", [(2, 1, 0), (1, 9, 0), (5, 3, 0), (120, 7, 0), (122, 40, 0), (244, 33, 0),
                                           (57, 30, 0), (113, 300, 0), (364, 2500, 0), (248, 50, 2), (124, 21, 3)])
def test_runs_equal_single_steps(nx, ny, variant, kind):
    flags = _flags(kind, nx, ny)
    one = _lattice(nx, ny, flags, 1, variant)
    say(f"[gpu] d2q9 runs {nx}x{ny} {kind} variant={variant}")
    for n in (1, 2, 3, 4, 7, 8, 50):
        one.step(n)
    m = np.ones((ny, nx), bool) if flags is None else flags == 0
    f_ref, sums_ref = one.get_f()[:, m], _sums(one, 75)
    for most in (2, 4):
        lat = _lattice(nx, ny, flags, most, variant)
        lat.step(75)
        f = lat.get_f()[:, m]
        # scattered lid sites can drive a run to infinity: a NaN's bits are not compared
        assert np.all((f.view(np.uint32) == f_ref.view(np.uint32)) | (np.isnan(f) & np.isnan(f_ref))), most
        assert _sums(lat, 75) == sums_ref, most
        lat.close()
    one.close()
