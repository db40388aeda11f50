"""Plans at the edge of the static scratch of fm_solve_static (host code)."""
import ctypes as C

import numpy as np
import pytest

import workloads as W

SCRATCH = 64 << 20


@pytest.fixture(scope="module")
def lib():
    import os
    from paper_2607_05929_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2607_05929_amd import build as _b
        _b.build()
    return binding.lib()


# grids whose workspace is within 2 KB of the scratch: the descriptors of the
# transforms may not outgrow it (conditions: two faces per component and axis)
@pytest.mark.parametrize("n,scheme,finite,bc", [
    ((69, 33, 98), W.TETRA2, 1, [2, 1, 2, 2, 2, 2, 1, 2, 1, 1, 2, 2, 1, 2, 2, 1, 1, 2]),
    ((57, 48, 108), W.HEX1, 1, [0, 0, 1, 2, 1, 2, 0, 0, 2, 2, 2, 1, 0, 0, 1, 2, 2, 1])])
def test_static_scratch(lib, n, scheme, finite, bc):
    from paper_2607_05929_amd import binding
    prob = W.random_small_problem(np.random.default_rng(0), n=(4, 4, 4), scheme=scheme,
                                  bc=np.array(bc, dtype=np.int32).reshape(3, 3, 2))
    d = binding.plan_desc(prob, prec=W.FP32_MIXED)
    for i in range(3):
        d.n[i] = n[i]
    d.green, d.finite_strain, d.tol, d.max_iter = W.GREEN_2MU0 if scheme == W.TETRA2 else W.GREEN_B0, finite, 1e-6, 10
    d.aa_depth, d.aa_period, d.max_materials, d.with_state = 4, 3, 2, 0
    bytes_ = lib.fm_workspace_bytes(C.byref(d))
    assert SCRATCH - 4096 < bytes_ <= SCRATCH
