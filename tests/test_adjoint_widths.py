"""A gradient is the same bits whatever the checkpoint interval and the vector
width of the forward kernel: steps that write their moments (recomputed and
last stretches) round like those that do not."""
import numpy as np
import pytest

import paper_2409_16781_amd as lbm
from paper_2409_16781_amd import inputs

from gpu_util import kernel_variant, require_gpu, say

pytestmark = pytest.mark.gpu

STEPS = 30


def _gradient(shape, flags, every, variant=None, tune=False):
    torch = require_gpu()
    nz, ny, nx = shape
    with kernel_variant(variant):
        lat = lbm.Lattice(nx, ny, nz, 0.6, flags=flags)
    lat.set_force(1e-6, 2e-6, -1e-6)
    fx = inputs.uniform_noise(shape, 5e-6, 7).astype(np.float32)
    lat.set_force_field(torch.from_numpy(fx).cuda())
    lat.init_eq(torch.from_numpy(1.0 + inputs.uniform_noise(shape, 1e-3, 8)).cuda(),
                torch.from_numpy(inputs.uniform_noise((3,) + shape, 2e-2, 9)).cuda())
    if tune:
        lat.tune(2)
    J, g = lat.grad_outlet_flux_x(STEPS, every)
    g, used = g.cpu().numpy(), lat.query(0)
    lat.close()
    return J, g, used


# rows of the widest vectors, and odd ones that only one site a lane fits
@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("shape", [(10, 12, 16), (6, 10, 17)])
def test_gradient_bits_at_every_width_and_interval(shape, solids):
    nz, ny, nx = shape
    flags = inputs.sphere_flags(nx, ny, nz, 0.85, 21, rmin=1.5, rmax=2.5) if solids else None
    say(f"[gpu] gradient widths {shape} solids={solids}")
    J0, g0, _ = _gradient(shape, flags, STEPS, 3)
    variants = (1, 2, 3) if nx % 4 == 0 else (3,)
    for kw in [dict(variant=v) for v in variants] + [dict(), dict(tune=True)]:
        for every in (1, 4, 7, STEPS):
            J, g, used = _gradient(shape, flags, every, **kw)
            assert J == J0 and np.array_equal(g.view(np.uint32), g0.view(np.uint32)), (kw, every, used)
