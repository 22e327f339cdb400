"""The launch-shape tuner times the kernels that the lattice runs afterwards
(their names as the profiler reports them), and the cache policy of the pulls
reaches every kernel that has one."""
import os

import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

from paper_2409_16781_amd import inputs

from gpu_util import make_lattice, say

pytestmark = pytest.mark.gpu


def _cfg(shape=(16, 32, 64)):
    nz, ny, nx = shape
    return dict(name="tuner", shape=shape, tau=0.6, force=(1e-5, 0.0, 0.0), flags=inputs.random_flags(nx, ny, nz, 0.2, 11),
                rho=1.0 + inputs.uniform_noise(shape, 1e-3, 21), u=inputs.uniform_noise((3,) + shape, 3e-2, 22))


def _step_kernels(call):
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return {e.name for e in prof.events() if "step_vec<" in e.name}


# FP16 lattices of default width round the rest population once, tuned ones
# like their width's ordinary kernel; with solids each of the three widths has
# a kernel with cached and one with non-temporal pulls
@pytest.mark.parametrize("codec", ["f16", "f32", "bf16", "s16"])
def test_tuner_times_the_kernels_that_run(codec):
    lat = make_lattice(_cfg(), codec)
    say(f"[gpu] tuner {codec}")
    timed = _step_kernels(lambda: lat.tune(2))
    assert len(timed) == 6, timed
    ran = _step_kernels(lambda: (lat.step(3), lat.sync()))
    assert ran and ran <= timed, (ran, timed)
    lat.close()


def test_non_temporal_pulls_of_the_default_fp16_width():
    got = []
    for nt in ("0", "1"):
        os.environ["LB_PULL_NT"] = nt
        try:
            lat = make_lattice(_cfg(), "f16")
        finally:
            os.environ.pop("LB_PULL_NT", None)
        say(f"[gpu] fp16 default width LB_PULL_NT={nt}")
        assert lat.info["variant"] == 3 and lat.query(12) == int(nt)
        got.append((_step_kernels(lambda: (lat.step(6), lat.sync())), lat.get_f().tobytes()))
        lat.close()
    assert got[0][0].isdisjoint(got[1][0]), got[0][0]
    assert got[0][1] == got[1][1]
