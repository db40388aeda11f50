"""Matrix-core transforms (short and odd axes): the Green operator against the
oracle at the edges of their 16-row tiles and of the sizes they cover, and an
autotuned plan on them against the untuned one."""
import numpy as np
import pytest

import workloads as W
from gpu_util import rel_err, xyz_nodes_from_zyx, zyx_nodes_from_xyz
from oracle import fd
from oracle import solver as osolver

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2607_05929_amd import binding
    binding.lib()
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return binding


# half matrices of n / 2 + 1 rows: one tile up to n = 31, one row in the last
# tile at 32, 64, 96; the smallest axis (4); a long axis beside short ones
# (the plane kernel takes the longer of y and z); prime lengths; the largest
# half matrices of either precision (six tiles in FP32, four in FP64)
SHAPES = [(4, 5, 6), (31, 32, 33), (30, 4, 64), (5, 63, 65), (61, 7, 29), (96, 8, 5), (6, 5, 125), (125, 90, 4)]
PATTERNS = {"P": [W.P, W.P], "N": [W.N, W.N], "D": [W.D, W.D], "ND": [W.N, W.D], "DN": [W.D, W.N]}


def _bc(rng, pattern):
    bc = np.zeros((3, 3, 2), dtype=np.int32)
    for q in range(3):
        for i in range(3):
            bc[q, i] = PATTERNS[pattern if pattern in PATTERNS else list(PATTERNS)[rng.integers(5)]]
    return bc


def _green(B, prec, shape, bc, scheme):
    rng = np.random.default_rng(sum(shape))
    prob = W.random_small_problem(rng, n=shape, scheme=scheme, bc=bc)
    pl = osolver.Plan(prob)
    x = rng.standard_normal((3,) + tuple(v + 1 for v in shape))
    for q in range(3):
        fd.zero_dismissed(x[q], pl.exts[q])
    ref = -pl.green_apply(x)
    gp = B.Plan(prob, prec=prec)
    got = xyz_nodes_from_zyx(gp.apply_green(zyx_nodes_from_xyz(x)))
    gp.close()
    # rounding of sums of at most 96 terms per axis and direction, relative to
    # the largest value: FP64 6 * 96 * 1.1e-16, FP32 6 * 96 * 6e-8 at worst
    tol = 1e-11 if prec == W.FP64 else 3.5e-5
    print(f"green n={shape} prec={prec} err={rel_err(got, ref):.2e}", flush=True)
    assert rel_err(got, ref) < tol


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pattern", ["P", "N", "D", "ND", "DN", "mix"])
def test_green_matrix_tiles(B, prec, shape, pattern):
    _green(B, prec, shape, _bc(np.random.default_rng(3 * sum(shape)), pattern), W.TETRA2)


@pytest.mark.parametrize("shape", [(190, 4, 5), (4, 5, 190), (5, 160, 9)])
@pytest.mark.parametrize("pattern", ["N", "ND"])
def test_green_matrix_longest_fp32(B, shape, pattern):
    _green(B, W.FP32_MIXED, shape, _bc(np.random.default_rng(1), pattern), W.TETRA2)


def test_autotuned_matrix_plan(B):
    """Timing the axis passes writes over the matrix tables: the tuned plan has
    to solve as the untuned one does."""
    prob = W.random_rve(np.random.default_rng(8), 45, prec=W.FP64, tol=1e-8)
    a, b = B.Plan(prob), B.Plan(prob)
    b.autotune(n_iter=2)
    ra, rb = a.solve(), b.solve()
    a.close(), b.close()
    assert ra["iters"] == rb["iters"]
    # both stop at the same error of 1e-8; their iterates differ by rounding
    assert rel_err(rb["sig"], ra["sig"]) < 1e-9
