"""C0 Green operator with wavefront z passes: every transform kind along z at
pencil lengths of each kernel form (16, 32 and 64 lanes, one to twelve points
per lane), against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import fd, solver as osolver
from tests.gpu_util import rel_err, xyz_nodes_from_zyx, zyx_nodes_from_xyz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
@pytest.mark.parametrize("zkind", range(5))
@pytest.mark.parametrize("shape,xy", [((6, 5, 16), (1, 2)), ((9, 4, 24), (0, 1)), ((5, 6, 32), (3, 0)),
                                      ((17, 5, 48), (2, 4)), ((4, 9, 64), (0, 0)), ((5, 4, 96), (1, 3)),
                                      ((6, 7, 192), (4, 0))])
def test_c0_green_z_lengths(prec, zkind, shape, xy):
    from paper_2607_05929_amd import binding as B
    rng = np.random.default_rng(sum(shape) + zkind)
    prob = W.random_small_problem(rng, n=shape, scheme=zkind % 2, bc=W.normal_mixed_bc(xy + (zkind,)))
    prob.green = W.GREEN_C0
    pl = osolver.Plan(prob)
    x = rng.standard_normal((3,) + tuple(v + 1 for v in shape))
    for q in range(3):
        fd.zero_dismissed(x[q], pl.exts[q])
    ref = -pl.green_apply(x)
    gp = B.Plan(prob, prec=prec)
    got = xyz_nodes_from_zyx(gp.apply_green(zyx_nodes_from_xyz(x)))
    gp.close()
    e = rel_err(got, ref)
    print(f"c0 z shape={shape} xy={xy} z={zkind} prec={prec} err {e:.2e}", flush=True)
    # FFT rounding: a few unit round-offs per stage (6e-8, 1.1e-16)
    assert e < (1e-11 if prec == W.FP64 else 2e-5)


# the 512-point pencils (eight points per lane, in FP32 the pipelined kernel)
# of each kind: 512 cells periodic, 256 with one condition on both faces, 128
# with one on each; 320 points (five per lane) from 160 and 80 cells; real and
# complex columns (x or y periodic); more columns than one tile
@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
@pytest.mark.parametrize("nz,zkind", [(512, 0), (256, 1), (256, 2), (128, 3), (128, 4),
                                      (320, 0), (160, 1), (160, 2), (80, 3), (80, 4)])
@pytest.mark.parametrize("n0,n1,xy", [(5, 6, (1, 2)), (6, 5, (0, 3)), (4, 7, (4, 0)), (37, 4, (0, 0)), (41, 5, (3, 1))])
def test_c0_green_z_long(prec, nz, zkind, n0, n1, xy):
    from paper_2607_05929_amd import binding as B
    rng = np.random.default_rng(nz + 10 * zkind + n0)
    prob = W.random_small_problem(rng, n=(n0, n1, nz), scheme=(zkind + n0) % 2, bc=W.normal_mixed_bc(xy + (zkind,)))
    prob.green = W.GREEN_C0
    pl = osolver.Plan(prob)
    x = rng.standard_normal((3, n0 + 1, n1 + 1, nz + 1))
    for q in range(3):
        fd.zero_dismissed(x[q], pl.exts[q])
    ref = -pl.green_apply(x)
    gp = B.Plan(prob, prec=prec)
    got = xyz_nodes_from_zyx(gp.apply_green(zyx_nodes_from_xyz(x)))
    gp.close()
    e = rel_err(got, ref)
    print(f"c0 z n={n0}x{n1}x{nz} xy={xy} z={zkind} prec={prec} err {e:.2e}", flush=True)
    # as above: FFT rounding, a few unit round-offs per stage
    assert e < (1e-11 if prec == W.FP64 else 2e-5)
