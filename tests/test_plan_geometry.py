"""Kernel choice of plans (host code, no GPU): the engine's make_geometry,
compiled for the host with tests/host/geometry.hip, asked for descriptors."""
import os
import subprocess

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FACES = {"P": (W.P, W.P), "N": (W.N, W.N), "D": (W.D, W.D), "M": (W.N, W.D)}


@pytest.fixture(scope="module")
def geometry(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "geometry")
    # host code only: the kernels' fat binary and the matrix-core launchers
    # stay unresolved, nothing here reaches them
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-O1", "-std=c++17", "-w",
                    "-I", os.path.join(ROOT, "include"), "-o", exe, os.path.join(ROOT, "tests", "host", "geometry.hip"),
                    "-Wl,--unresolved-symbols=ignore-all"], check=True)

    def ask(n, prec, bc, scheme=W.TETRA2, green=W.GREEN_B0):
        """(on the matrix cores, kernel per component and pass) of a plan; bc:
        its conditions, or one of FACES per axis for every component."""
        bc = [f for _ in range(3) for c in bc for f in FACES[c]] if isinstance(bc, str) else np.asarray(bc).reshape(-1)
        line = " ".join(str(int(v)) for v in (*n, prec, scheme, green, *bc))
        out = subprocess.run([exe], input=line + "\n", capture_output=True, text=True, check=True).stdout
        head, rest = out.strip().split(" |")
        rc, mat = (int(v) for v in head.split())
        assert rc == 0, rest
        names = rest.split()
        return bool(mat), [names[7 * q:7 * q + 7] for q in range(3)]
    return ask


def test_wavefront_offsets(geometry):
    """The wavefront kernels stop where the buffers of their own pass reach
    4 GiB per component: here the z spectrum does, which only the split z
    passes of the C0 operator use."""
    n = (2000, 4096, 64)
    # reals of the z input and of the z spectrum, 8 bytes each
    assert 8 * 2001 * 4097 * 65 < 2 ** 32 <= 8 * 2001 * 4097 * 66
    c0 = W.normal_mixed_bc((1, 1, 0))
    for q in range(3):
        assert geometry(n, W.FP64, "NNP")[1][q][2] == "64x1"
        assert geometry((2000, 2048, 64), W.FP64, c0, green=W.GREEN_C0)[1][q][5:] == ["64x1", "64x1"]
    # (the component with the longest spectrum: cosines along x and y)
    assert ["-", "-"] in [k[5:] for k in geometry(n, W.FP64, c0, green=W.GREEN_C0)[1]]


# one short axis (fewer than 16 cells) without a wavefront kernel: plans whose
# planes of complex data are few, or fill a second round in FP64, stay on the
# axis passes; their neighbours, and grids with a longer or a second such
# axis, run on the matrix cores
@pytest.mark.parametrize("n,pattern,fp32,fp64", [
    ((6, 64, 64), "PPP", 0, 0), ((6, 64, 64), "PPD", 0, 0), ((6, 64, 64), "DPP", 1, 1), ((6, 64, 64), "DNN", 1, 1),
    ((4, 64, 32), "PPM", 0, 0), ((5, 96, 96), "PPP", 0, 0), ((5, 64, 96), "PPP", 0, 0), ((15, 64, 32), "PPP", 0, 0),
    ((17, 64, 32), "PPP", 1, 1), ((10, 64, 48), "PPP", 1, 1), ((11, 48, 64), "PPP", 1, 1), ((11, 16, 32), "PPP", 1, 1), ((11, 16, 64), "PPP", 0, 0),
    ((6, 64, 57), "PPP", 1, 1), ((6, 32, 32), "PPP", 1, 1), ((64, 7, 64), "PPP", 1, 1), ((64, 64, 7), "PPP", 1, 1),
    ((96, 64, 5), "DPP", 1, 0), ((96, 9, 32), "NPP", 1, 0), ((96, 64, 5), "PPP", 1, 1), ((96, 48, 10), "DPP", 1, 0), ((96, 16, 9), "DPP", 1, 1),
    ((64, 64, 5), "DPP", 1, 1), ((96, 64, 17), "DPP", 1, 1), ((96, 5, 96), "DNN", 1, 1), ((96, 11, 13), "DPP", 1, 1)])
def test_short_axes(geometry, n, pattern, fp32, fp64):
    assert geometry(n, W.FP32_MIXED, pattern)[0] == bool(fp32)
    assert geometry(n, W.FP64, pattern)[0] == bool(fp64)


# the lines of cubes with wavefront kernels throughout, and the longest axis
# of either precision on the matrix cores
@pytest.mark.parametrize("n,prec,pattern,mat", [
    ((64, 64, 64), W.FP64, "DNN", 1), ((96, 96, 96), W.FP64, "DNN", 0), ((96, 96, 96), W.FP32_MIXED, "MMM", 0),
    ((95, 95, 95), W.FP64, "DNN", 1), ((48, 48, 48), W.FP64, "PPP", 1), ((64, 64, 64), W.FP32_MIXED, "PPP", 0),
    ((191, 5, 6), W.FP32_MIXED, "NNN", 1), ((192, 5, 6), W.FP32_MIXED, "NNN", 0),
    ((127, 5, 6), W.FP64, "NNN", 1), ((128, 5, 6), W.FP64, "NNN", 0),
    ((6, 127, 5), W.FP32_MIXED, "PPP", 1), ((6, 128, 5), W.FP32_MIXED, "PPP", 0),
    ((6, 95, 5), W.FP64, "PPP", 1), ((6, 96, 5), W.FP64, "PPP", 0)])
def test_matrix_lengths(geometry, n, prec, pattern, mat):
    assert geometry(n, prec, pattern)[0] == bool(mat)
