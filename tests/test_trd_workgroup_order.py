"""CPU replay of the tridiagonalisation (stage 1 of the eigensolver, eig.hip).

The kernels and their launch loop are taken from the source file as they are
and compiled for the host: the threads of a workgroup run as fibers that meet
at the barriers and at the wave reductions, the workgroups of a launch one
after another, in ascending or in descending order.  Nothing orders the
workgroups of a launch on the GPU, so that both orders have to give the same
bits: a word that one workgroup writes and another reads in the same launch is
seen old in one order and new in the other."""

import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

import host_lanes
from host_lanes import CLANG, CSRC, between

SHIM = host_lanes.SHIM + r"""
struct GemmDesc {
    int m, n, k, transa = 0, transb = 0;
    const double *A, *B, *Cin = nullptr;
    double* C;
    long long lda, ldb, ldc, ldcin = 0;
    double alpha = 1.0, beta = 0.0;
};
static hipError_t gemm(const GemmDesc& g, hipStream_t) {   // as the loop below uses it: C = Cin - A B^T
    if (g.transa || !g.transb || g.alpha != -1.0 || g.beta != 1.0 || g.Cin != g.C || g.ldcin != g.ldc) std::abort();
    for (int j = 0; j < g.n; ++j)
        for (int i = 0; i < g.m; ++i) {
            double s = 0.0;
            for (int k = 0; k < g.k; ++k) s += g.A[i + k * g.lda] * g.B[j + k * g.ldb];
            g.C[i + j * g.ldc] -= s;
        }
    return hipSuccess;
}
template <class T>
static hipError_t fill_matrix(int m, int n, T* Z, long long ld, long long, int, double diag, double off, hipStream_t) {
    for (int j = 0; j < n; ++j)
        for (int i = 0; i < m; ++i) Z[i + j * ld] = i == j ? diag : off;
    return hipSuccess;
}
template <class T>
T* carve(char*& p, size_t count) {
    T* r = reinterpret_cast<T*>(p);
    p += ((count * sizeof(T) + 255) / 256) * 256;
    return r;
}
"""

TAIL = r"""
extern "C" int trd(int n, double* A, double* d_out, double* e_out, double* tau_out, long work_bytes, char* work,
                   int descending) {
    g_descending = descending;
    if ((long)syevd_work_bytes(n) > work_bytes) return -1;
    std::vector<double> zbuf((size_t)n * n);
    double* Z = zbuf.data();
    const long long lda = n, ldz = n;
    hipStream_t st = 0;
    // as in syevd
    %(setup)s
    %(loop)s
    (void)Z; (void)ldz; (void)err;
    std::copy(d, d + n, d_out);
    std::copy(e, e + n - 1, e_out);
    std::copy(tau, tau + n - 1, tau_out);
    %(unscale)s
    return p - work > (long)syevd_work_bytes(n) ? -2 : %(refused)s;
}
"""


def source():
    src = open(os.path.join(CSRC, "eig.hip")).read()
    common = open(os.path.join(CSRC, "common.hpp")).read()
    consts = "".join(re.findall(r"^constexpr int k(?:TB|BT|FT|ET|MaxG)\b.*\n", src, flags=re.M))
    hh = between(common, "__device__ __forceinline__ void householder", "// Number of XCDs")
    kernels = between(src, "struct TrdArgs {", "// T factors (compact WY)")
    sizes = between(src, "static int factor_ld", "// Eigen-decomposition of the symmetric")
    setup = between(src, "    char* p = work;", "    // --- Stage 1")
    loop = between(src, "    // --- Stage 1", "    // --- Stage 2")
    loop = host_lanes.launches(loop)
    unscale = "if (*scale > 0.0) for (int i = 0; i < n; ++i) { d_out[i] /= *scale; if (i + 1 < n) e_out[i] /= *scale; }"
    return "\n".join([SHIM, "namespace {", consts, hh, kernels, "}", sizes,
                      TAIL % {"setup": setup, "loop": loop, "unscale": unscale,
                              "refused": "*scale == 0.0 ? 1 : 0"}])


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++")
    d = tmp_path_factory.mktemp("trd")
    (d / "trd.cpp").write_text(source())
    r = subprocess.run([CLANG, "-O1", "-std=c++17", "-w", "-shared", "-fPIC", "-o", str(d / "trd.so"), str(d / "trd.cpp")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(str(d / "trd.so"))


def tridiagonalise(lib, A, descending, status=0):
    n = A.shape[0]
    F = np.array(A, order="F")
    d, e, tau = np.zeros(n), np.zeros(max(n - 1, 1)), np.zeros(max(n - 1, 1))
    work = np.full((32 << 20) // 8, np.nan)
    ptr = lambda x: x.ctypes.data_as(ctypes.c_void_p)
    rc = lib.trd(n, ptr(F), ptr(d), ptr(e), ptr(tau), ctypes.c_long(work.nbytes), ptr(work), descending)
    assert rc == status
    return d, e[:n - 1], tau[:n - 1], F


def symmetric(n, seed):
    B = np.random.default_rng(seed).standard_normal((n, n))
    return (B + B.T) / 2


# One row group, two, and several with a ragged last one; one panel and several.
@pytest.mark.parametrize("n", [2, 33, 65, 129, 200])
def test_any_order_of_workgroups_gives_the_same_bits(lib, n):
    A = symmetric(n, n)
    up = tridiagonalise(lib, A, 0)
    down = tridiagonalise(lib, A, 1)
    for x, y in zip(up, down):
        assert np.array_equal(x, y)
    d, e = up[:2]
    T = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
    # Backward error of a Householder reduction, a modest multiple of n eps ||A||.
    w, ref = np.linalg.eigvalsh(T), np.linalg.eigvalsh(A)
    assert np.abs(w - ref).max() <= 4 * n * np.finfo(float).eps * np.abs(ref).max()


# The product with the raw column makes x^T A x of the order of ||A||^3: whatever
# the norm, the reduction is that of the matrix of norm about 1.  Scaling by a
# power of two is exact (no entry here is subnormal), so T and the reflectors keep
# their bits.
@pytest.mark.parametrize("exponent", [-1000, -480, -350, -33, -32, -31, 0, 31, 32, 33, 350, 480, 1000])
def test_scaled_matrices(lib, exponent):
    n = 60
    A = symmetric(n, 7)
    d0, e0, tau0, _ = tridiagonalise(lib, A, 0)
    d, e, tau, _ = tridiagonalise(lib, np.ldexp(A, exponent), 0)
    assert np.array_equal(d, np.ldexp(d0, exponent)) and np.array_equal(e, np.ldexp(e0, exponent))
    assert np.array_equal(tau, tau0)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("at", [(0, 0), (40, 3), (69, 69)])
def test_non_finite_matrices_are_refused(lib, bad, at):
    # The rank of a NaN eigenvalue among others is no permutation, and the merges
    # index by it: nothing that is not finite may come out of this stage.
    A = symmetric(70, 3)
    A[at] = A[at[::-1]] = bad
    d, e, tau, F = tridiagonalise(lib, A, 0, status=1)
    assert not d.any() and not e.any() and not tau.any() and np.all(np.isfinite(F))
