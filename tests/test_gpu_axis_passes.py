"""The axis passes (fm_wave.h, fm_pass.h) at short and odd pencils.  On small
grids those lengths run on the matrix cores; here one axis is too long for
them, so that the whole plan stays on the axis passes: pencils of 16 and 32
lanes, the 96- and 192-point kernels specialised by kind, and the generic LDS
passes, on each axis, against the oracle."""
import zlib

import numpy as np
import pytest

import workloads as W
from oracle import fd
from oracle import solver as osolver
from tests.gpu_util import xyz_nodes_from_zyx, zyx_nodes_from_xyz
from tests.test_gpu_parity import BC_PATTERNS

pytestmark = pytest.mark.gpu

# 16-, 32-, 48-, 64-, 96-, 128-, 192- and 320-point pencils (n = 8, 16, 24, 48,
# 64, 96, 128, 160; DFT and the doubled lengths) on every axis, then lengths with radices 3, 5, 7, 11, 13 and a
# prime one (generic passes)
SHAPES = [(48, 16, 256), (24, 256, 8), (16, 256, 48), (96, 8, 256), (8, 256, 24), (256, 48, 24), (256, 16, 96),
          (256, 96, 16), (256, 24, 48), (6, 96, 256), (5, 256, 96),
          (64, 5, 256), (256, 64, 5), (5, 256, 64), (128, 256, 5), (256, 5, 128), (6, 128, 256),
          (160, 256, 5), (256, 160, 4), (4, 256, 160),
          (256, 7, 11), (13, 256, 9), (9, 15, 256), (29, 256, 6), (256, 12, 61), (5, 200, 14)]


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pattern", ["P", "N", "D", "ND", "DN", "mix"])
def test_green_on_axis_passes(prec, shape, pattern):
    from paper_2607_05929_amd import binding as B
    rng = np.random.default_rng(zlib.crc32(repr((shape, pattern)).encode()))
    names = list(BC_PATTERNS)
    bc = np.zeros((3, 3, 2), dtype=np.int32)
    for q in range(3):
        for i in range(3):
            bc[q, i] = BC_PATTERNS[pattern if pattern != "mix" else names[(q + 2 * i) % len(names)]]
    prob = W.random_small_problem(rng, n=shape, bc=bc, scheme=(SHAPES.index(shape) + len(pattern) + prec) % 2)
    pl = osolver.Plan(prob)
    x = rng.standard_normal((3,) + tuple(v + 1 for v in shape))
    for q in range(3):
        fd.zero_dismissed(x[q], pl.exts[q])
    ref = -pl.green_apply(x)
    gp = B.Plan(prob, prec=prec)
    assert not gp.matrix_transforms()
    got = xyz_nodes_from_zyx(gp.apply_green(zyx_nodes_from_xyz(x)))
    gp.close()
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"axis passes n={shape} {pattern} scheme={prob.scheme} prec={prec} err={err:.2e}", flush=True)
    # rounding, in units u of the precision: one for each stage of the six
    # transforms of a point (at most log2 L = 10 radix-2 stages each) and five
    # for the Green factor; in FP64 the reference too has these, and the
    # cosines near pi / 2 in its denominators an error of n u each, squared in
    # two of the axes
    u = 2.0 ** -53 if prec == W.FP64 else 2.0 ** -24
    assert err < (65 * u if prec == W.FP32_MIXED else (2 * 65 + 8 * max(shape)) * u)
