"""Stress-divergence tiles of solves with internal variables: the law
evaluated in the tile (J2 among elastic materials), stresses read from the
stress pass (crystal plasticity), and a batch of both with an elastic solve."""
import zlib

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import rel_err, xyz_nodes_from_zyx, zyx_nodes_from_xyz
from oracle import fd
from oracle import solver as osolver
from oracle.laws import MaterialSet
from tests.test_gpu_parity import _bc_pattern

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2607_05929_amd import binding
    binding.lib()
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return binding


# several x-y tiles with ragged edges, one-column and one-layer tiles, and a
# grid large enough for tiles of several layers (the carried faces)
@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
@pytest.mark.parametrize("scheme", [W.HEX1, W.TETRA2])
@pytest.mark.parametrize("pattern,shape", [("P", (40, 17, 9)), ("mix", (30, 6, 16)), ("mixwrap", (62, 13, 33)),
                                           ("P", (66, 60, 50)), ("mix", (63, 70, 41))])
def test_state_law_tiles(B, prec, scheme, pattern, shape):
    rng = np.random.default_rng(zlib.crc32(f"{shape}{pattern}{scheme}".encode()))
    prob = W.random_small_problem(rng, n=shape, scheme=scheme, law="j2", bc=_bc_pattern(rng, pattern))
    prob.materials = list(prob.materials) + [W.mat_iso(1.3, 0.7), W.mat_cubic(2.0, 1.1, 0.8, np.array([0.5, 0.5, 0.5, 0.5]))]
    prob.mat_id = rng.integers(0, len(prob.materials), np.asarray(prob.mat_id).shape).astype(np.int32)
    pl = osolver.Plan(prob)
    uf = 1e-3 * rng.standard_normal((3,) + tuple(v + 1 for v in shape))
    for q in range(3):
        fd.zero_dismissed(uf[q], pl.exts[q])
    step = prob.steps[0]
    mats = MaterialSet(prob.materials, np.asarray(prob.mat_id).transpose(2, 1, 0))
    gu = pl.grad(uf) + pl.grad(pl.ustar(step.c, step.G, step.H))
    sig, _ = mats.stress(0.5 * (gu + np.swapaxes(gu, -1, -2)), mats.init_state(pl.nppv, pl.n), step.dt)
    ref = pl.div(sig)
    gp = B.Plan(prob, prec=prec)
    D, err, macro = gp.residual(zyx_nodes_from_xyz(uf), step)
    gp.close()
    D = xyz_nodes_from_zyx(D)
    kept = np.stack(pl.kept)
    ms = sig.mean(axis=(0, 1, 2, 3))
    mref = np.array([ms[i, j] for (i, j) in osolver.VOIGT])
    e, em = rel_err(D[kept], ref[kept]), rel_err(macro, mref)
    print(f"state tiles shape={shape} {pattern} scheme={scheme} prec={prec} D {e:.2e} macro {em:.2e}", flush=True)
    # FP32: D sums stresses rounded to FP32 (6e-8 times the stencil's cancellation)
    assert np.all(D[~kept] == 0.0)
    assert e < (1e-10 if prec == W.FP64 else 5e-5)
    assert em < (1e-12 if prec == W.FP64 else 1e-5)


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
def test_batch_of_all_stress_sources(B, prec):
    """Elastic, J2 and crystal-plasticity members in one batch stop where they
    stop alone."""
    probs = []
    for k, law in enumerate(["cubic", "j2", "cp", "iso", "j2"]):
        p = W.random_small_problem(np.random.default_rng(40 + k), n=(9 + k, 8, 7), scheme=k % 2, law=law, tol=1e-5)
        p.prec = prec
        probs.append(p)
    alone = [B.solve(p, prec=prec) for p in probs]
    both = B.batch_solve(probs, prec=prec, fields=True)
    for a, b in zip(alone, both):
        assert list(a["iters"]) == list(b["iters"])
        # the same arithmetic but for the order of the partial sums (FP64)
        assert rel_err(b["sig"], a["sig"]) < (1e-9 if prec == W.FP64 else 1e-5)
