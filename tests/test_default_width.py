"""The vector width a lattice gets by default (storage, size, solids) changes
no bit of its state: it equals that of the widest vectors, which every lattice
of a length they fit used to have, and runs of the one-site kernel equal its
steps taken one by one."""
import os

import numpy as np
import pytest
import torch

import paper_2409_16781_amd as lbm
from paper_2409_16781_amd import inputs

from gpu_util import make_lattice, say

pytestmark = pytest.mark.gpu


def _cfg(shape, solids, force=(1e-5, 0.0, -2e-5)):
    nz, ny, nx = shape
    return dict(name="width", shape=shape, tau=0.6, force=force,
                flags=inputs.random_flags(nx, ny, nz, 0.2, 11) if solids else None,
                rho=1.0 + inputs.uniform_noise(shape, 1e-3, 21), u=inputs.uniform_noise((3,) + shape, 3e-2, 22))


def _run(cfg, codec, variant, n=12):
    lat = make_lattice(cfg, codec, variant)
    lat.step(n)
    rho, u = lat.step_macros(3)
    got = lat.get_f(), rho.cpu().numpy(), u.cpu().numpy(), lat.info["variant"]
    lat.close()
    return got


# 2^16 is the bound of FP32's narrowest vectors, 2^18 that of 16-bit ones with
# solids; nx of 8, a multiple of 8 that is no power of two, and a wave's width
@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("codec", ["f32", "f16", "bf16", "s16"])
@pytest.mark.parametrize("shape", [(3, 5, 8), (16, 64, 64), (17, 64, 64), (32, 64, 128), (33, 64, 128), (7, 9, 120)])
def test_default_width_keeps_the_state(shape, codec, solids):
    cfg = _cfg(shape, solids)
    say(f"[gpu] default width {shape} {codec} solids={solids}")
    f, rho, u, v = _run(cfg, codec, None)
    g, rho1, u1, v1 = _run(cfg, codec, 1)
    assert v1 == 1
    m = np.ones(shape, bool) if cfg["flags"] is None else cfg["flags"] == 0
    assert np.array_equal(f[:, m], g[:, m]), v
    assert np.array_equal(rho, rho1) and np.array_equal(u, u1), v


def test_a_force_field_takes_the_widest_vectors_while_it_is_set():
    cfg = _cfg((12, 16, 32), True)
    lat = make_lattice(cfg, "f32")
    narrow = lat.info["variant"]
    lat.step(70)
    lat.set_force_field(torch.zeros(cfg["shape"], dtype=torch.float32, device="cuda"))
    assert narrow == 3 and lat.query(0) == 1
    lat.step(70)
    lat.set_force_field(None)
    assert lat.query(0) == narrow
    lat.step(70)
    assert np.all(np.isfinite(lat.sums(210)))
    lat.close()


@pytest.mark.parametrize("codec", ["f32", "f16", "bf16", "s16"])
@pytest.mark.parametrize("shape", [(3, 5, 7), (47, 75, 101)])
def test_runs_of_the_one_site_kernel_equal_single_steps(shape, codec):
    cfg = _cfg(shape, True)
    a, b = make_lattice(cfg, codec, 0), make_lattice(cfg, codec, 0)
    say(f"[gpu] one-site runs {shape} {codec}")
    a.step(67)
    a.step(6)
    for _ in range(73):
        b.step(1)
    m = cfg["flags"] == 0
    assert np.array_equal(a.get_f()[:, m], b.get_f()[:, m])
    assert np.array_equal(a.sums(73).view(np.uint64), b.sums(73).view(np.uint64))
    a.close()
    b.close()
