"""GPU parity of the symmetric eigensolver of Zolo-SVD (Algorithm 2's
H = V diag(S) V^T; zolo_dsyevd through the C ABI): Householder
tridiagonalisation, divide and conquer, back-transformation.

Eigenvalues are compared with LAPACK (NumPy) and with the oracle's own
Jacobi eigensolver, eigenvectors through the residual ||A Z - Z diag(w)|| and
orthogonality (the paper's OrthR = ||I - V^T V||_F / n < 1.0e-15, Section
4.1), and, where the spectrum is known exactly, the eigenvalues with it."""

import numpy as np
import pytest

from oracle import dense as od
from paper_1806_06204_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def z():
    import torch
    from paper_1806_06204_amd import zolo
    assert torch.cuda.is_available()
    h = zolo.Zolo()
    yield h
    h.close()


def dev(x):
    from paper_1806_06204_amd import zolo
    return zolo.to_device(x)


def check(z, A, tol_res=1e-14):
    n = A.shape[0]
    w, Z = z.syevd(dev(A))
    Z = Z.cpu().numpy()
    nrm = np.linalg.norm(A, 2) if n > 1 else abs(A[0, 0])
    nrm = max(nrm, 1e-300)
    res = np.linalg.norm(A @ Z - Z * w) / (nrm * np.sqrt(n))
    orth = np.linalg.norm(Z.T @ Z - np.eye(n)) / n
    ev = np.max(np.abs(w - np.linalg.eigvalsh(A)[::-1])) / nrm
    print(f"  n={n}: res={res:.2e} OrthR={orth:.2e} eig err={ev:.2e}", flush=True)
    assert np.all(np.diff(w) <= 0)
    assert res <= tol_res and orth <= 1e-15 and ev <= 1e-14
    return w, Z


@pytest.mark.parametrize("n", [1, 2, 3, 31, 32, 33, 64, 65, 127, 200, 333])
def test_random_symmetric(z, n):
    rng = np.random.default_rng(900 + n)
    B = rng.standard_normal((n, n))
    check(z, (B + B.T) / 2)


@pytest.mark.parametrize("n", [129, 513, 1025])
def test_merges_past_a_wave(z, n):
    # Merges whose pole count leaves a remainder over the 64 lanes that share
    # a root, on a spectrum that deflates little and on one that deflates a lot.
    rng = np.random.default_rng(950 + n)
    V = W.haar(n, n, 80 + n)
    for s in (rng.standard_normal(n), np.repeat(rng.standard_normal(n // 3 + 1), 3)[:n]):
        check(z, (V * s) @ V.T)


@pytest.mark.parametrize("n", [128, 130, 256, 257, 258, 386])
def test_back_transformation_block_edges(z, n):
    # Reflector counts just below, at and past 128 (one factor in LDS) and 256
    # (one block), even and odd leading dimensions.  The eigenvalues are
    # settled before the back-transformation: residual and orthogonality judge it.
    rng = np.random.default_rng(970 + n)
    B = rng.standard_normal((n, n))
    A = (B + B.T) / 2
    w, Z = z.syevd(dev(A))
    Z = Z.cpu().numpy()
    assert np.linalg.norm(A @ Z - Z * w) <= 1e-14 * np.linalg.norm(A, 2) * np.sqrt(n)
    assert np.linalg.norm(Z.T @ Z - np.eye(n)) <= 1e-15 * n


def test_graded_and_clustered_spectra(z):
    # The spectra H has in Zolo-SVD: log-spaced over 16 decades, and clusters
    # of nearly equal eigenvalues (many deflations in the merges).
    n = 300
    V = W.haar(n, n, 77)
    for lam in (np.logspace(0, -16, n), np.repeat([1.0, 1e-3, 1e-9], n // 3),
                np.concatenate([np.ones(150), np.full(150, 0.5)])):
        A = (V * lam) @ V.T
        A = (A + A.T) / 2
        w, _ = check(z, A)
        assert np.max(np.abs(w - np.sort(lam)[::-1])) <= 1e-14


def test_matches_oracle_jacobi(z):
    # Against the oracle's own eigensolver (pinned to 50-digit mpmath): the
    # eigenvalues, and the eigenvectors up to sign (distinct eigenvalues).
    rng = np.random.default_rng(5)
    n = 48
    B = rng.standard_normal((n, n))
    A = (B + B.T) / 2
    lo, Vo = od.jacobi_eigh(A)
    w, Z = z.syevd(dev(A))
    Z = Z.cpu().numpy()
    assert np.max(np.abs(w - lo)) <= 1e-13 * np.max(np.abs(lo))
    s = np.sign(np.sum(Z * Vo, axis=0))
    assert np.max(np.abs(Z * s - Vo)) <= 1e-12


def test_tridiagonal_input_and_lower_triangle_only(z):
    # A tridiagonal matrix is its own reduction (all reflectors trivial), and
    # only the lower triangle is read.
    n = 150
    rng = np.random.default_rng(8)
    d, e = rng.standard_normal(n), rng.standard_normal(n - 1)
    T = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
    check(z, T)
    Tl = np.tril(T) + np.triu(np.full((n, n), 7.0), 1)    # garbage above the diagonal
    w, Z = z.syevd(dev(Tl))
    assert np.max(np.abs(w - np.linalg.eigvalsh(T)[::-1])) <= 1e-14 * np.linalg.norm(T, 2)


@pytest.mark.parametrize("n", [2, 60, 257])
def test_only_the_lower_triangle_is_read(z, n):
    rng = np.random.default_rng(1100 + n)
    B = rng.standard_normal((n, n))
    A = (B + B.T) / 2
    w0, Z0 = check(z, A)
    w, Z = z.syevd(dev(np.tril(A) + np.triu(np.full((n, n), 7.0), 1)))
    assert np.array_equal(w, w0) and np.array_equal(Z.cpu().numpy(), Z0)


# A power of two on the matrix is the same power of two on its eigenvalues, bit
# for bit, and leaves the eigenvectors alone; orders around the 520 pinned words of
# the handle.
@pytest.mark.parametrize("n,exponent", [(60, -1000), (60, -480), (60, -350), (60, 350), (60, 480), (60, 1000),
                                        (511, -400), (512, 400), (519, 400), (520, -400)])
def test_scaled_by_powers_of_two(z, n, exponent):
    rng = np.random.default_rng(1200 + n)
    B = rng.standard_normal((n, n))
    A = (B + B.T) / 2
    w0, Z0 = z.syevd(dev(A))
    Z0 = Z0.cpu().numpy()
    assert np.linalg.norm(A @ Z0 - Z0 * w0) <= 1e-14 * np.linalg.norm(A, 2) * np.sqrt(n)
    w, Z = z.syevd(dev(np.ldexp(A, exponent)))
    assert np.array_equal(w, np.ldexp(w0, exponent))
    assert np.array_equal(Z.cpu().numpy(), Z0)


@pytest.mark.parametrize("exponent", [-480, -350, 350, 480])
def test_svd_scaled_by_powers_of_two(z, exponent):
    m, n = 150, 70
    A, _, s, _ = W.svd_matrix(m, n, 20.0, 61, 62)
    U0, S0, V0, i0 = z.svd(dev(A), alpha=1.0, l=0.04)
    U, S, V, info = z.svd(dev(np.ldexp(A, exponent)), alpha=float(np.ldexp(1.0, exponent)), l=0.04)
    assert info["status"] == i0["status"] == 0
    assert np.array_equal(S, np.ldexp(S0, exponent)) and np.abs(S0 - s).max() <= 1e-13
    assert np.array_equal(U.cpu().numpy(), U0.cpu().numpy()) and np.array_equal(V.cpu().numpy(), V0.cpu().numpy())


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_is_refused(z, bad):
    A = np.eye(40)
    A[7, 5] = A[5, 7] = bad
    from paper_1806_06204_amd.zolo import ZoloError
    with pytest.raises(ZoloError, match="code 2"):
        z.syevd(dev(A))
    check(z, np.eye(40))                         # the handle goes on working


# Orders just past the lines where a wave of the tridiagonalisation's product takes
# two and four columns, odd: leading dimension, last group of columns and pair loads.
@pytest.mark.parametrize("n", [2051, 4099])
def test_columns_per_wave(z, n):
    import torch
    g = torch.Generator().manual_seed(n)
    B = torch.randn((n, n), generator=g, dtype=torch.float64)
    A = (B + B.T) / 2
    print(f"  n={n}: solving", flush=True)
    w, Z = z.syevd(A.cuda())
    Z = Z.cpu()
    nrm = max(abs(w[0]), abs(w[-1]))
    assert np.all(np.diff(w) <= 0)
    assert float(torch.linalg.norm(A @ Z - Z * torch.from_numpy(w))) <= 1e-14 * nrm * np.sqrt(n)
    assert float(torch.linalg.norm(Z.T @ Z - torch.eye(n, dtype=torch.float64))) <= 1e-15 * n


def test_exact_spectrum_n4096(z):
    # H = V diag(sigma) V^T with sigma log-spaced from 1 to 1e-16 (the H of
    # the kappa = 1e16 workload at n = 4096): eigenvalues against sigma.
    n = 4096
    V = W.haar(n, n, 2003)
    sig = W.logspaced_sigma(n, 1e16)
    import torch
    Vt = torch.from_numpy(V)
    H = ((Vt * torch.from_numpy(sig)) @ Vt.T).numpy()
    H = (H + H.T) / 2
    print("  n=4096 exact spectrum: solving", flush=True)
    w, Z = z.syevd(dev(H))
    err = np.max(np.abs(w - sig))
    Zt = torch.from_numpy(Z.cpu().numpy())
    orth = float(torch.linalg.norm(Zt.T @ Zt - torch.eye(n, dtype=torch.float64))) / n
    res = float(torch.linalg.norm(torch.from_numpy(H) @ Zt - Zt * torch.from_numpy(w))) / np.sqrt(n)
    print(f"  max |w - sigma| = {err:.2e}, OrthR = {orth:.2e}, res = {res:.2e}", flush=True)
    assert err <= 1e-14 and orth <= 1e-15 and res <= 1e-14
