"""Per-step totals of FP32 lattices against exact sums of the stored state:
weak flows (moments far below one quantum of a whole-lattice split), ordinary
ones, moments beyond the split's range, and non-finite states."""
import os

import numpy as np
import pytest
import torch

import paper_2409_16781_amd as lbm

from gpu_util import FP64_SUM_TOL, exact_state_totals, require_gpu, say

pytestmark = pytest.mark.gpu


def _with_env(env, make):
    os.environ.update(env)
    try:
        return make()
    finally:
        for k in env:
            os.environ.pop(k, None)


# A uniform flow: every site has the same moments, so every site's loss adds
# up (1e-14: populations are multiples of 2^-80 and finer, below the quanta of
# a split sized for the whole lattice, 2^-69 at 64^3).  The sums of the absolute
# values of the stored populations scale the bound of the FP64 summation trees.
@pytest.mark.parametrize("u", [1e-14, 1e-5, 0.03])
@pytest.mark.parametrize("two,inplace", [("2", False), ("0", False), ("2", True)])
@pytest.mark.parametrize("shape", [(64, 64, 64), (13, 1100, 128)])
def test_box_totals_are_the_sums_of_the_state(shape, two, inplace, u):
    require_gpu()
    nz, ny, nx = shape
    lat = _with_env({"LB_TWO_STEP": two}, lambda: lbm.Lattice(nx, ny, nz, 0.7, inplace=inplace))
    uu = torch.empty((3,) + shape, dtype=torch.float64, device="cuda")
    for c, f in enumerate((1.0, -0.3, 0.07)):
        uu[c] = f * u
    lat.init_eq(None, uu)
    say(f"[gpu] totals of a uniform flow {shape} LB_TWO_STEP={two} inplace={inplace} u={u}")
    for n in (2, 1):
        lat.step(n)
        g = lat.get_f().astype(np.float64)
        exact, scale = exact_state_totals(g, np.ones(shape, bool))
        got = lat.sums(1)[0]
        tol = FP64_SUM_TOL * scale
        tol[0] += 2.0 ** -52 * exact[0]  # both masses are rounded once more, with the number of sites in them
        assert np.all(np.abs(got - exact) <= tol), (n, got - exact, tol)
    lat.close()


@pytest.mark.parametrize("u", [1e-14, 0.03])
@pytest.mark.parametrize("most", ["1", "2", "4"])
def test_d2q9_totals_are_the_sums_of_the_state(most, u):
    require_gpu()
    nx, ny = 260, 1050
    lat = _with_env({"LB_STEPS2D": most}, lambda: lbm.Lattice2D(nx, ny, 0.7))
    uu = torch.empty((2, ny, nx), dtype=torch.float64, device="cuda")
    uu[0], uu[1] = u, -0.3 * u
    lat.init_eq(None, uu)
    lat.step(4)
    g = lat.get_f().astype(np.longdouble)
    cx = np.array([0, 1, -1, 0, 0, 1, 1, -1, -1])[:, None, None]
    cy = np.array([0, 0, 0, 1, -1, 1, -1, 1, -1])[:, None, None]
    got = lat.sums(1)[0]
    say(f"[gpu] totals of a uniform flow {nx}x{ny} LB_STEPS2D={most} u={u}")
    for k, c in enumerate((1, cx, cy)):
        exact, scale = float((c * g).sum()), float(np.abs(c * g).sum())
        n = float(nx * ny) if k == 0 else 0.0
        assert abs(got[k] - (n + exact)) <= FP64_SUM_TOL * scale + 2.0 ** -52 * n, k
    lat.close()


# Mass deviations of 1e4 a site are beyond the two parts' exact range: the
# totals are then ordinary FP64 sums, and the tolerance theirs.  tau = inf:
# the state only streams.
@pytest.mark.parametrize("two", ["2", "0"])
def test_totals_beyond_the_split_range(two):
    require_gpu()
    shape = (9, 33, 96)
    lat = _with_env({"LB_TWO_STEP": two}, lambda: lbm.Lattice(shape[2], shape[1], shape[0], float("inf")))
    rho = 1.0 + 1e4 * torch.rand(shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    lat.init_eq(rho, None)
    lat.step(2)
    exact, scale = exact_state_totals(lat.get_f().astype(np.float64), np.ones(shape, bool))
    assert np.all(np.abs(lat.sums(1)[0] - exact) <= FP64_SUM_TOL * scale + 2.0 ** -53 * np.abs(exact))
    lat.close()


@pytest.mark.parametrize("steps", [1, 2])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_states_are_reported(value, steps):
    require_gpu()
    lat = lbm.Lattice(64, 64, 64, 0.7)
    assert lat.query(13) == 2
    rho = torch.ones((64, 64, 64), dtype=torch.float64, device="cuda")
    rho[5, 6, 7] = value
    lat.init_eq(rho, None)
    lat.step(steps)
    with pytest.raises(lbm.LBError):
        lat.sums(1)
    lat.close()
