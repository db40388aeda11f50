"""Matrix-core transforms on the GPU at the longest axes they take, with the
HEX1 operator (whose result hangs on few modes), and the rounding of their
products."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import xyz_nodes_from_zyx, zyx_nodes_from_xyz
from tests.test_transform_lanes import PAIRS, U, _error, _plan, rounding

pytestmark = pytest.mark.gpu


def _green(n, prec, scheme, kinds, seed):
    """(case, input, result); the plan is asserted to be on the matrix cores."""
    from paper_2607_05929_amd import binding as B
    case = (n, prec, scheme, 0, kinds, 0, seed)
    pl = _plan(case)
    prob = W.random_small_problem(np.random.default_rng(0), n=n, scheme=scheme,
                                  bc=np.array([[PAIRS[k] for k in row] for row in kinds], dtype=np.int32))
    prob.lambda0, prob.mu0 = 1.25, 0.75
    x = np.random.default_rng(seed).standard_normal((3,) + tuple(v + 1 for v in n))
    if prec == W.FP32_MIXED:
        x = x.astype(np.float32).astype(np.float64)
    for q in range(3):
        x[q][~pl.kept[q]] = 0.0
    gp = B.Plan(prob, prec=prec)
    assert gp.matrix_transforms()
    got = xyz_nodes_from_zyx(gp.apply_green(zyx_nodes_from_xyz(x)))
    gp.close()
    return case, x, got


def _held(case, x, got):
    err, tol = _error(case, x, got)
    print(f"matrix n={case[0]} scheme={case[2]} prec={case[1]} kinds={case[4]} err={err:.2f} u of {tol:.1f}", flush=True)
    assert err < tol


# six tiles in FP32 (191 cells), four in FP64 and for planes of complex data in
# FP32 (127), three for those in FP64 (95): odd lengths whose last tile is full
# and whose results past the row end in its padding; kinds: 0 periodic, 1 N/N,
# 2 D/D, 3 N/D, 4 D/N
@pytest.mark.parametrize("scheme", [W.HEX1, W.TETRA2])
@pytest.mark.parametrize("axis", range(3))
@pytest.mark.parametrize("n,prec,kind,others", [
    (191, W.FP32_MIXED, 1, (3, 2)), (191, W.FP32_MIXED, 2, (1, 4)), (191, W.FP32_MIXED, 3, (4, 1)),
    (191, W.FP32_MIXED, 4, (2, 3)), (127, W.FP64, 1, (4, 3)), (127, W.FP64, 2, (3, 1)),
    (125, W.FP64, 3, (1, 2)), (125, W.FP64, 4, (2, 2)), (127, W.FP32_MIXED, 0, (0, 3)), (127, W.FP32_MIXED, 0, (1, 0)),
    (127, W.FP32_MIXED, 0, (0, 0)), (95, W.FP64, 0, (0, 2)), (95, W.FP64, 0, (0, 0)), (127, W.FP64, 0, (4, 1))])
def test_longest_axes(n, prec, kind, others, axis, scheme):
    size, row = [5, 6, 7], [0, 0, 0]
    size[axis], row[axis] = n, kind
    rest = [a for a in range(3) if a != axis]
    for a, k in zip(rest, others):
        row[a] = k
    _held(*_green(tuple(size), prec, scheme, [row] * 3, n + axis))


# tile edges as in test_gpu_matrix.py, every kind on every axis over the components
@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
@pytest.mark.parametrize("shift", range(4))
@pytest.mark.parametrize("n", [(4, 5, 6), (31, 32, 33), (30, 4, 64), (5, 63, 65), (61, 7, 29), (96, 8, 5), (6, 5, 125),
                               (125, 90, 4)])
def test_hex1_tile_edges(n, shift, prec):
    kinds = [[1 + (shift + q + a * (1 + q)) % 4 for a in range(3)] for q in range(3)]
    _held(*_green(n, prec, W.HEX1, kinds, 7 * shift + n[0]))


@pytest.mark.parametrize("n", [(12, 180, 12), (180, 12, 12), (12, 12, 180), (60, 60, 60), (12, 100, 51)])
def test_rounding_of_the_products(n):
    """As on the host: below the geometric mean of what several chains of
    partial sums and one chain leave (TETRA2, FP32, all kinds but the periodic
    one, averaged)."""
    e2 = []
    for k in range(1, 5):
        case, x, got = _green(n, W.FP32_MIXED, W.TETRA2, [[k] * 3] * 3, k)
        ref = -_plan(case).green_apply(x)
        e2.append((np.linalg.norm(got - ref) / np.linalg.norm(ref) / U[W.FP32_MIXED]) ** 2)
    err = np.mean(e2) ** 0.5
    print(f"rounding n={n}: {err:.2f} u, chains {rounding(n):.2f}, one chain {rounding(n, ones=True):.2f}", flush=True)
    assert err < (rounding(n) * rounding(n, ones=True)) ** 0.5
