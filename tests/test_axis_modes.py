"""The modes of an axis of uneven cells (spectral_modes.cpp), compiled alone
for the CPU: what is found is an eigenvector basis, and what is not found is
said."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1409_0001_amd", "csrc")

SHIM = r"""
#include "spectral_modes.cpp"
#include <algorithm>
extern "C" int modes(int n, double* d, const double* e, double* z) {
    std::vector<double> dd(d, d + n), ee(e, e + n - 1);
    cgd::Rotations r;
    if (!cgd::tridiagonal_modes(dd, ee, r)) return 0;
    std::copy(dd.begin(), dd.end(), d);
    for (int k = 0; k < n * n; ++k) z[k] = k % (n + 1) == 0;
    size_t q = 0;
    for (const auto& s : r.sweeps) {
        if (s.lo < 0 || s.count < 1 || s.lo + s.count >= n) return -1;
        for (int k = s.lo; k < s.lo + s.count; ++k, q += 2)
            for (int i = 0; i < n; ++i) {
                const double u = z[k * n + i], v = z[(k + 1) * n + i];
                z[k * n + i] = r.cs[q] * u + r.cs[q + 1] * v;
                z[(k + 1) * n + i] = r.cs[q] * v - r.cs[q + 1] * u;
            }
    }
    if (q != r.cs.size()) return -1;
    // the same from the groups, as a device thread per column steps through them
    cgd::RotationGroups g;
    cgd::group_rotations(r, g);
    constexpr int L = cgd::RotationGroups::kLanes;
    for (int i = 0; i < n; ++i) {
        std::vector<double> col(n, 0.0);
        col[i] = 1.0;
        const double* cs = g.cs.data();
        for (const auto& s : g.groups) {
            if (s.lo < 0 || s.rows < 2 || s.lo + s.rows > n || s.count % cgd::RotationGroups::kGroupSteps) return -2;
            double u[L] = {col[s.lo]};
            for (int t = 0; t < s.count; ++t) {
                double v = col[s.lo + std::min(t + 1, s.rows - 1)];
                for (int j = 0; j < L; ++j, cs += 2) {
                    const double o = cs[0] * u[j] + cs[1] * v;
                    u[j] = cs[0] * v - cs[1] * u[j];
                    v = o;
                }
                const int r = t + 1 - L;
                if (r >= 0 && r < s.rows) col[s.lo + r] = v;
            }
        }
        if (cs != g.cs.data() + g.cs.size()) return -3;
        for (int k = 0; k < n; ++k)
            if (std::fabs(col[k] - z[k * n + i]) > 1e-15) return -4;
    }
    return 1;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("modes")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def _modes(lib, d, e):
    n = len(d)
    d, e = np.array(d, np.float64), np.array(e, np.float64)
    z = np.zeros((n, n))
    p = ctypes.POINTER(ctypes.c_double)
    ok = lib.modes(n, d.ctypes.data_as(p), e.ctypes.data_as(p), z.ctypes.data_as(p))
    assert ok >= 0, ok  # (sweeps within the matrix, all rotations used, the groups the same)
    return bool(ok), d, z


def _laplacian(h):
    g = np.concatenate([[0.0], 2.0 / (h[:-1] + h[1:]), [0.0]])
    return (g[:-1] + g[1:]) / h, -g[1:-1] / np.sqrt(h[:-1] * h[1:])


@pytest.mark.parametrize("n", [2, 3, 17, 64, 200])
@pytest.mark.parametrize("ratio", [1.0, 1.05, 1.5])
def test_modes_are_an_eigenvector_basis(lib, n, ratio):
    """Orthonormal to 1e-13 n, and the residual of every pair within 1e-14 n
    of the matrix's norm."""
    d, e = _laplacian(ratio ** np.minimum(np.arange(n), 60.0))
    ok, lam, z = _modes(lib, d, e)
    assert ok
    A = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
    assert np.abs(z @ z.T - np.eye(n)).max() <= 1e-13 * n
    assert np.abs(A @ z.T - z.T * lam).max() <= 1e-14 * n * np.abs(A).max()
    assert np.abs(np.sort(lam) - np.linalg.eigvalsh(A)).max() <= 1e-14 * n * np.abs(A).max()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("where", ["diagonal", "off-diagonal"])
def test_what_is_not_found_is_said(lib, bad, where):
    d, e = _laplacian(1.02 ** np.arange(20.0))
    (d if where == "diagonal" else e)[7] = bad
    assert not _modes(lib, d, e)[0]


def test_overflow_is_said(lib):
    """Entries near the largest float64: the rotations' products overflow."""
    d, e = _laplacian(np.ones(30))
    assert not _modes(lib, d * 5e307, e * 5e307)[0]
