"""The matrix-core transforms without a GPU: fm_mat.hip compiled for the host,
its wavefronts run in lockstep (tests/host/lanes), launched by the engine's own
plan, tables and work lists.  Every buffer lies between pages without access,
so an index out of range ends the run; LDS and spectral planes start as NaN, so
a value that is read but not written shows in the result; and each node's
displacement has to take its increment once."""
import os
import subprocess

import numpy as np
import pytest

import workloads as W
from oracle import dt, fd, green
from oracle import solver as osolver
from tests.gpu_util import xyz_nodes_from_zyx

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host", "lanes")
# (component q, axis i) -> conditions of the two faces
PAIRS = [(W.P, W.P), (W.N, W.N), (W.D, W.D), (W.N, W.D), (W.D, W.N)]
U = {W.FP64: 2.0 ** -53, W.FP32_MIXED: 2.0 ** -24}


@pytest.fixture(scope="module")
def lanes(tmp_path_factory):
    tmp = str(tmp_path_factory.mktemp("lanes"))
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    kernels = subprocess.Popen([os.path.join(rocm, "llvm", "bin", "clang++"), "-std=c++17", "-O2", "-w", "-I", HOST, "-c",
                                "-o", tmp + "/lanes.o", os.path.join(HOST, "lanes.cpp")])
    subprocess.run([os.path.join(rocm, "bin", "hipcc"), "--offload-host-only", "-O1", "-std=c++17", "-w", "-I",
                    os.path.join(ROOT, "include"), "-c", "-o", tmp + "/engine.o", os.path.join(HOST, "transforms.hip")],
                   check=True)
    assert kernels.wait() == 0
    subprocess.run([os.path.join(rocm, "bin", "hipcc"), "-o", tmp + "/transforms", tmp + "/engine.o", tmp + "/lanes.o",
                    "-Wl,--unresolved-symbols=ignore-all"], check=True)

    def run(cases):
        """[input x, result] or None where the plan is refused, per case (n,
        prec, scheme, green, kind[q][axis] (indices into PAIRS), terms, seed)."""
        text = "".join(" ".join(str(int(v)) for v in (*n, prec, scheme, green,
                                                      *[f for row in kinds for k in row for f in PAIRS[k]], terms, seed))
                       + "\n" for n, prec, scheme, green, kinds, terms, seed in cases)
        path = tmp + "/fields.bin"
        p = subprocess.run([tmp + "/transforms", path], input=text, capture_output=True, text=True)
        lines = p.stdout.splitlines()
        assert p.returncode == 0 and "FAULT" not in p.stdout and lines[-1] == "done", "\n".join(lines[-2:]) + p.stderr
        data, out, at, line = np.fromfile(path), [], 0, 0
        for n, *_ in cases:
            line += 1
            if lines[line] == "refused":
                line += 1
                out.append(None)
                continue
            nn = 3 * (n[0] + 1) * (n[1] + 1) * (n[2] + 1)
            f = data[at:at + 2 * nn].reshape(2, 3, n[2] + 1, n[1] + 1, n[0] + 1)
            out.append([xyz_nodes_from_zyx(v) for v in f])
            at += 2 * nn
        assert at == data.size
        return out
    return run


def _plan(case):
    n, prec, scheme, green, kinds, terms, seed = case
    bc = np.array([[PAIRS[k] for k in row] for row in kinds], dtype=np.int32)
    prob = W.random_small_problem(np.random.default_rng(0), n=n, scheme=scheme, bc=bc)
    prob.green, prob.lambda0, prob.mu0 = green, 1.25, 0.75
    return osolver.Plan(prob)


def _error(case, x, got):
    """Relative L2 error in units u, and what it may be: four times what the
    oracle's own transforms leave when their values are rounded to FP32
    (few modes carry a HEX1 result, and hit or miss), or what ``rounding``
    expects with the Anderson terms of a node; in FP64 the oracle's own error,
    its cosines near pi / 2 being off by n u each, squared in two axes."""
    pl, prec = _plan(case), case[1]
    ref = -pl.green_apply(x)
    norm = np.linalg.norm(ref) * U[prec]
    err = np.linalg.norm(got - ref) / norm
    tol = 4 * (rounding(case[0]) ** 2 + case[5]) ** 0.5
    if prec == W.FP64:
        return err, tol + 130 + 8 * max(case[0])
    return err, max(tol, 4 * np.linalg.norm(green_fp32(pl, x) - ref) / norm)


def green_fp32(pl, x):
    """Minus the oracle's Green operator with the values after each transform,
    and the denominators, rounded to FP32."""
    def fp32(a):
        return a.astype(np.complex64 if np.iscomplexobj(a) else np.float32)
    out = np.zeros_like(x)
    for q in range(3):
        kinds, a = pl.kinds[q], fp32(x[q])
        for i in range(3):
            a = fp32(dt.forward_1d(a, kinds[i], i))
        null = green.null_mask(kinds, pl.n, pl.scheme)
        den = green.denominator(kinds, pl.n, q, pl.scheme, pl.h, pl.lam0, pl.mu0, pl.green)
        a = fp32(np.where(null, 0, a / np.where(null, 1, den).astype(np.float32)))
        for i in (2, 1, 0):
            a = fp32(dt.inverse_1d(a, kinds[i], i, pl.n[i]))
        out[q] = a.real
        fd.zero_dismissed(out[q], pl.exts[q])
    return out


def rounding(n, ones=False):
    """RMS rounding error of the operator relative to its result, in units u:
    a sum of N = n / 2 + 1 random terms in c chains (eight from N = 49 on, else
    four) leaves the partial sums of each, of mean square k terms at step k,
    rounded with a mean square of u^2 / 6 of theirs, so N / 6 c of the
    result's; a point passes two such sums per axis, and about 2.5 more for
    what is stored between them and the Green factor.  ones: one chain."""
    e = 2.5
    for v in n:
        terms = v // 2 + 1
        e += 2 * terms / 6 / (1 if ones else 8 if terms > 48 else 4)
    return e ** 0.5


def _periodic(kinds, axes):
    return [[0 if a in axes else kinds[q][a] for a in range(3)] for q in range(3)]


def _edge_cases(prec):
    """Every kind of transform on every axis at lengths around the edges of the
    16-row tiles and of the sizes the kernels take, beside two short axes;
    with one, two and three periodic axes."""
    longest, pair = (191, 127) if prec == W.FP32_MIXED else (127, 95)
    lengths = [4, 5, 6, 29, 30] + [n for n in range(31, longest + 1) if n % 32 in (31, 0)] + [longest - 1]
    cases, seed = [], 0
    for n in lengths:
        for axis in range(3):
            for kind in range(5):
                seed += 1
                rng = np.random.default_rng(seed)
                size = [int(v) for v in rng.integers(4, 8, 3)]
                size[axis] = n
                kinds = rng.integers(1, 5, (3, 3))
                kinds[:, axis] = kind
                if kind == 0 and n <= pair:
                    kinds = np.array(_periodic(kinds, [axis, (axis + 1 + seed % 2) % 3][:1 + seed % 3] if seed % 4 else [0, 1, 2]))
                cases.append((tuple(size), prec, seed % 2, seed // 2 % 2, kinds.tolist(), 1 + seed % 4, seed))
    return cases


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_MIXED])
def test_accesses_at_tile_edges(lanes, prec):
    cases = _edge_cases(prec)
    refused = 0
    for case, fields in zip(cases, lanes(cases)):
        if fields is None:
            refused += 1
            continue
        err, tol = _error(case, *fields)
        assert err < tol, (case, err, tol)
    # (in FP64 some long pencils with a prime factor past five are no plan's)
    assert refused == 0 if prec == W.FP32_MIXED else refused < len(cases) // 4


# a plane with both axes at four to six tiles, several row tiles per
# wavefront, and the narrow tails of both; planes of complex data both ways
@pytest.mark.parametrize("case", [
    ((5, 160, 190), W.FP32_MIXED, W.TETRA2, 0, [[1, 1, 1], [2, 3, 4], [3, 4, 2]], 1, 1),
    ((4, 125, 90), W.FP64, W.HEX1, 1, [[1, 4, 1], [2, 3, 4], [3, 2, 2]], 2, 2),
    ((6, 127, 97), W.FP32_MIXED, W.HEX1, 0, [[0, 0, 0]] * 3, 1, 3),
    ((7, 65, 90), W.FP64, W.TETRA2, 0, [[0, 3, 0], [0, 1, 0], [0, 4, 0]], 3, 4),
    ((9, 127, 63), W.FP32_MIXED, W.TETRA2, 1, [[1, 0, 0], [2, 0, 0], [4, 0, 0]], 2, 5),
    ((63, 31, 33), W.FP32_MIXED, W.TETRA2, 0, [[0, 0, 3], [0, 0, 1], [0, 0, 2]], 4, 6)])
def test_planes(lanes, case):
    fields, = lanes([case])
    err, tol = _error(case, *fields)
    assert err < tol, (err, tol)


@pytest.mark.parametrize("n", [(12, 180, 12), (180, 12, 12), (12, 12, 180), (60, 60, 60), (12, 100, 51)])
def test_chains_of_partial_sums(lanes, n):
    """The rounding of the products stays that of several chains of partial
    sums: below the geometric mean of theirs and of a single chain's (TETRA2,
    all kinds but the periodic one, averaged)."""
    cases = [(n, W.FP32_MIXED, W.TETRA2, 0, [[k] * 3] * 3, 1, k) for k in range(1, 5)]
    e2 = []
    for case, (x, got) in zip(cases, lanes(cases)):
        ref = -_plan(case).green_apply(x)
        e2.append((np.linalg.norm(got - ref) / np.linalg.norm(ref) / U[W.FP32_MIXED]) ** 2)
    assert np.mean(e2) ** 0.5 < (rounding(n) * rounding(n, ones=True)) ** 0.5
