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
