"""What a plan reports of its transforms: the path it runs on, and per-kernel
times that are zero for the passes it does not have."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _check(pl, mat):
    assert pl.matrix_transforms() == mat
    t = pl.profile(n_iter=3)
    pl.reset()
    for k in pl.KERNELS:
        assert (t[k] == 0.0) == (mat and k in ("y_fwd", "y_inv")), (k, t)


# an odd grid; one with wavefront kernels throughout and an axis past the matrix cores' sizes
@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
@pytest.mark.parametrize("shape,mat", [((21, 19, 23), True), ((16, 24, 256), False)])
def test_profile_and_path(prec, shape, mat):
    from paper_2607_05929_amd import binding as B
    bc = np.full((3, 3, 2), W.D, dtype=np.int32)
    prob = W.random_small_problem(np.random.default_rng(3), n=shape, bc=bc)
    pl = B.Plan(prob, prec=prec)
    _check(pl, mat)
    pl.autotune(n_iter=2)
    # (a tuned plan keeps whichever was faster; there is nothing to keep without the matrix cores)
    kept = pl.matrix_transforms()
    assert mat or not kept
    _check(pl, kept)
    pl.close()
