"""Calls of one step on small lattices (whose launch sums its own totals) give
the state, totals and fields of runs."""
import numpy as np
import pytest

from paper_2409_16781_amd import inputs

from gpu_util import make_lattice, say

pytestmark = pytest.mark.gpu


# one workgroup, a few, 64 (the most that sum their own totals) and more, at
# one site a lane (FP32) and two (16-bit)
@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("codec", ["f32", "f16", "bf16", "s16"])
@pytest.mark.parametrize("shape", [(2, 4, 8), (5, 6, 32), (16, 32, 32), (16, 33, 32), (32, 32, 32), (33, 32, 32)])
def test_single_steps_equal_a_run(shape, codec, solids):
    nz, ny, nx = shape
    cfg = dict(name="lone", shape=shape, tau=0.6, force=(1e-5, 0.0, -2e-5),
               flags=inputs.random_flags(nx, ny, nz, 0.2, 11) if solids else None,
               rho=1.0 + inputs.uniform_noise(shape, 1e-3, 21), u=inputs.uniform_noise((3,) + shape, 3e-2, 22))
    a, b = make_lattice(cfg, codec), make_lattice(cfg, codec)
    say(f"[gpu] lone steps {shape} {codec} solids={solids} grid={a.info['grid']}")
    for _ in range(12):
        a.step(1)
    ra, ua = a.step_macros(1)
    b.step(10)
    rb, ub = b.step_macros(3)
    m = np.ones(shape, bool) if cfg["flags"] is None else cfg["flags"] == 0
    assert np.array_equal(a.get_f()[:, m], b.get_f()[:, m])
    assert np.array_equal(a.sums(13).view(np.uint64), b.sums(13).view(np.uint64))
    assert np.array_equal(ra.cpu().numpy(), rb.cpu().numpy()) and np.array_equal(ua.cpu().numpy(), ub.cpu().numpy())
    a.close()
    b.close()
