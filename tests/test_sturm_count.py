"""The eigenvalue count behind the tridiagonal eigensolves (csrc/sturm.h), compiled
for the host, against numpy: decoupled blocks with the shift on an eigenvalue of a
leading block, random matrices, and every remainder of the four-row groups."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#define __host__
#define __device__
#include "%s"
extern "C" int count(const double *al, const double *be, int m, double x) {
    double b2[1024];
    for (int i = 0; i < m; ++i) b2[i] = ed::sturm_b2(i + 1 < m ? be[i] : 0.0);
    return ed::sturm_count(al, b2, m, x);
}
"""


@pytest.fixture(scope="module")
def count(tmp_path_factory):
    d = tmp_path_factory.mktemp("sturm")
    src, lib = d / "sturm.cpp", d / "sturm.so"
    src.write_text(SRC % os.path.join(ROOT, "paper_1004_3354_amd", "csrc", "sturm.h"))
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wno-unknown-pragmas", str(src), "-o", str(lib)],
                   check=True)
    f = ctypes.CDLL(str(lib)).count
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_double]

    def call(al, be, x):
        al, be = np.ascontiguousarray(al, dtype=np.float64), np.ascontiguousarray(np.append(be, 0.0), dtype=np.float64)
        return f(al.ctypes.data, be.ctypes.data, len(al), x)

    return call


def _check(count, al, be, xs):
    """Counts lie between the number of eigenvalues below x and at most x, up to the
    rounding of the matrix (norm 1)."""
    w = np.linalg.eigvalsh(np.diag(al) + np.diag(be, 1) + np.diag(be, -1))
    tol = 16 * len(al) * 2.0 ** -53
    for x in xs:
        c = count(al, be, float(x))
        assert np.sum(w < x - tol) <= c <= np.sum(w <= x + tol), (len(al), x, c, w)


@pytest.mark.parametrize("coupling", [0.0, 1e-200, 1e-30])
@pytest.mark.parametrize("m", range(1, 24))
def test_decoupled_blocks(count, m, coupling):
    """Blocks of one, two and three rows with eigenvalues that are exact in binary,
    (nearly) uncoupled, in random order; x on each eigenvalue and between them."""
    rng = np.random.default_rng(m)
    for _ in range(40):
        al, be = [], []
        while len(al) < m:
            kind = int(rng.integers(3))
            a = float(rng.integers(-4, 5)) / 8
            if kind == 0:
                al += [a]
                be += [coupling]
            elif kind == 1:                      # a -+ 1/4
                al += [a, a]
                be += [0.25, coupling]
            else:                                # a, a -+ 1/4 sqrt(2)
                al += [a, a, a]
                be += [0.25, 0.25, coupling]
        al, be = np.array(al[:m]), np.array(be[:m - 1])
        grid = np.arange(-8, 9) / 8
        _check(count, al, be, np.concatenate([grid, grid + 1 / 16, grid + 2.0 ** -40]))


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6, 8, 9, 31, 120, 257, 600])
def test_random_matrices(count, m):
    """Diagonals and couplings over many orders of magnitude."""
    rng = np.random.default_rng(100 + m)
    for _ in range(6):
        al = rng.uniform(-0.5, 0.5, m) * 10.0 ** rng.uniform(-12, 0, m)
        be = 0.25 * 10.0 ** rng.uniform(-25, 0, max(m - 1, 0))
        w = np.linalg.eigvalsh(np.diag(al) + np.diag(be, 1) + np.diag(be, -1))
        _check(count, al, be, np.concatenate([rng.uniform(-1, 1, 30), w[::max(1, m // 20)], al[:20], [0.0]]))
