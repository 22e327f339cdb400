"""lb_step_noalloc up to the size its scratch holds: 131 584 step workgroups of
64 bytes (split totals: 128) and a slot of the reduction per 256 of them."""
import os

import numpy as np
import pytest

import paper_2409_16781_amd as lbm

from gpu_util import kernel_variant, require_gpu, say

pytestmark = pytest.mark.gpu


# one site per lane (odd rows): 257 x 512 x 256 sites in 131 584 workgroups
@pytest.mark.parametrize("codec,two", [("f16", "1"), ("f32", "0"), ("f32", "2")])
def test_noalloc_accepts_what_fits(codec, two):
    require_gpu()
    os.environ["LB_TWO_STEP"] = two
    try:
        with kernel_variant(None):
            a, b = (lbm.Lattice(257, 512, 256, 0.8, codec=codec) for _ in range(2))
    finally:
        os.environ.pop("LB_TWO_STEP", None)
    assert a.info["grid"] == 131584
    say(f"[gpu] noalloc limit {codec} LB_TWO_STEP={two}")
    for lat in (a, b):
        lat.init_eq()
    assert lbm.lib().lb_step_noalloc(a.handle, 3) == lbm.LB_OK, lbm.last_error()
    b.step(3)
    assert np.array_equal(a.sums(3).view(np.uint64), b.sums(3).view(np.uint64))
    a.close()
    b.close()
