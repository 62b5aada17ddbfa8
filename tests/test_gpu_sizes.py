"""Kernels at the sizes where their work splits: tile and wave edges,
remainders, the smallest and the largest of a variant's range."""

import numpy as np
import pytest

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


@pytest.mark.parametrize("m,n", [(1, 1), (15, 3), (16, 16), (17, 5), (65, 63), (130, 65), (300, 257)])
def test_alpha_estimate(z, m, n):
    # 1.01 sigma_max by power iteration on 16-row workgroups and 64 column
    # groups; a gap of 2 leaves (1/2)^40 after ten steps.
    s = np.concatenate([[1.0], np.linspace(0.5, 0.1, n - 1)]) * 3.7
    A, _, _, _ = W.svd_matrix(m, n, 10.0, 60 + m, 70 + n, sigma=s)
    _, _, info = z.pd(dev(A))
    assert info["status"] == 0
    assert abs(info["alpha"] / (1.01 * 3.7) - 1.0) <= 1e-9


def check_qr(z, m, n, pivots, batch, seed):
    """QR of [Y; p I] (or of Y): the bounds of the structured-QR block tests,
    and R against LAPACK up to row signs."""
    rng = np.random.default_rng(seed)
    Y = rng.standard_normal((batch, m, n)) / np.sqrt(m)
    import torch
    Q, R = z.structured_qr(torch.from_numpy(Y).to("cuda"), pivots, form_q=True)
    Q, R = Q.cpu().numpy(), R.cpu().numpy()
    for b in range(batch):
        S = np.vstack([Y[b], pivots[b] * np.eye(n)]) if pivots else Y[b]
        assert np.linalg.norm(Q[b].T @ Q[b] - np.eye(n)) <= 1e-14 * n, b
        assert np.linalg.norm(Q[b] @ R[b] - S) <= 1e-14 * n * np.linalg.norm(S), b
        assert np.array_equal(np.tril(R[b], -1), np.zeros((n, n)))
        Rl = np.linalg.qr(S, mode="r")
        s = np.sign(np.diag(R[b])) * np.sign(np.diag(Rl))
        assert np.abs(R[b] * s[:, None] - Rl).max() <= 1e-12 * np.abs(Rl).max(), b


# Live rows (m + 64, or m without pivots) around each shape of the
# register-leaf panel: 256, 512, 1024 rows in one workgroup, then several
# workgroups with a ragged last slab; columns around the 16-column leaves and
# the 64-column panels; a single column; the shortest panels.
@pytest.mark.parametrize("m,n,batch,stacked", [
    (1, 1, 2, True), (5, 3, 1, True), (17, 17, 2, False), (33, 31, 1, True), (64, 64, 1, False), (65, 65, 2, True),
    (192, 64, 2, True), (193, 79, 1, True), (256, 20, 1, False), (257, 64, 1, False), (448, 64, 1, True),
    (449, 96, 2, True), (960, 65, 1, True), (1024, 64, 1, False), (1025, 64, 3, False), (1217, 130, 1, True),
    (2111, 64, 2, True)])
def test_panel_shapes(z, m, n, batch, stacked):
    pivots = [0.7 / (b + 1) for b in range(batch)] if stacked else None
    check_qr(z, m, n, pivots, batch, 31 * m + n)


@pytest.mark.parametrize("m,n,batch,stacked", [
    (70, 18, 1, False), (64, 33, 2, True), (250, 47, 1, False), (255, 49, 1, True), (400, 63, 2, False),
    (512, 31, 1, False), (704, 65, 2, True), (769, 40, 9, False), (769, 64, 1, False), (900, 100, 1, True)])
def test_panel_widths_and_placement(z, m, n, batch, stacked):
    # One to four leaves, whole and cut short, in one workgroup and in several;
    # more matrices than XCDs.
    pivots = [0.7 / (b + 1) for b in range(batch)] if stacked else None
    check_qr(z, m, n, pivots, batch, 17 * m + n)


def test_panel_beyond_the_tallest_shape(z):
    # 16 matrices of 33 000 rows: more 2048-row slabs than the GPU holds at once.
    check_qr(z, 33000, 66, None, 16, 5)


def test_panel_zero_and_graded_columns(z):
    # A zero column (no reflector), equal columns, and columns over 140 decades.
    import torch
    rng = np.random.default_rng(9)
    Y = rng.standard_normal((1, 300, 70))
    Y[0, :, 5] = 0.0
    Y[0, :, 20] = Y[0, :, 19]
    Y[0] *= np.power(10.0, -np.linspace(0.0, 140.0, 70))
    Q, R = z.structured_qr(torch.from_numpy(Y).to("cuda"), None, form_q=True)
    Q, R = Q[0].cpu().numpy(), R[0].cpu().numpy()
    assert np.linalg.norm(Q.T @ Q - np.eye(70)) <= 1e-14 * 70
    d = np.linalg.norm(Q @ R - Y[0], axis=0)
    assert np.all(d <= 1e-14 * 70 * np.linalg.norm(Y[0], axis=0))


def test_reflector_of_one_column(z):
    # Q[0] = 1 - tau = alpha / beta of a column [alpha; x], tau = (|alpha| + |col|) / |col|
    # in [1, 2].  With x^2 exact the norm is off by 1.5 u (its argument and the root),
    # which tau takes at most half of, and the sum and the quotient by u each.
    import torch
    rng = np.random.default_rng(77)
    u = 2.0 ** -53
    worst = 0.0
    for _ in range(200):
        Y = np.empty((16, 2, 1))
        Y[:, 0, 0] = 2.0 ** rng.uniform(-30.0, 2.0, 16) * rng.choice([-1.0, 1.0], 16)
        Y[:, 1, 0] = np.round(rng.uniform(0.5, 1.0, 16) * 2 ** 24) / 2 ** 24
        Q, _ = z.structured_qr(torch.from_numpy(Y).to("cuda"), None, form_q=True)
        al, x = Y[:, 0, 0].astype(np.longdouble), Y[:, 1, 0].astype(np.longdouble)
        tau = 1 + np.abs(al) / np.sqrt(al * al + x * x)
        worst = max(worst, float(np.max(np.abs((1 - Q.cpu().numpy()[:, 0, 0].astype(np.longdouble)) / tau - 1))))
    print(f"  largest error of tau: {worst / u:.3f} u")
    assert worst <= 2.75 * u * (1 + 1e-3)


@pytest.mark.parametrize("m,n", [(1024 - 64, 130), (1985, 70), (2048 - 64, 200), (2100, 100)])
def test_batched_panels_one_workgroup(z, m, n):
    # The many-matrix call's panels: one workgroup up to 2048 live rows, more
    # past that; one stream and several give the same bits.
    A, U, s, V = W.svd_matrix(m, n, 1e3, 600 + m, 700 + n)
    mats = [dev(A), dev(A[:200, :50] + np.eye(200, 50)), dev(A)]
    Q1, H1, i1 = z.pd_batched(mats, alphas=[1.0, 3.0, 1.0], ls=[1e-3, 1e-3, 1e-3], batch_streams=1)
    Q2, H2, i2 = z.pd_batched(mats, alphas=[1.0, 3.0, 1.0], ls=[1e-3, 1e-3, 1e-3], batch_streams=3)
    for a, b in zip(Q1 + H1, Q2 + H2):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
    assert i1[0]["kinds"][0] == "Q"
    Hx = (V * s) @ V.T
    for k in (0, 2):
        assert np.linalg.norm(H1[k].cpu().numpy() - Hx) <= 1e-12 * np.linalg.norm(Hx)
        Q = Q1[k].cpu().numpy()
        assert np.linalg.norm(Q.T @ Q - np.eye(n)) <= 1e-13 * np.sqrt(n)


# Orders around the 16-row steps and the 64-column blocks of the Cholesky and
# of the triangular inverse, in both precisions.
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 33, 48, 63, 64, 65, 100, 127, 129, 257])
def test_cholesky_and_inverse_edges(z, n, dtype):
    import torch
    rng = np.random.default_rng(40 + n)
    X = rng.standard_normal((3, 2 * n + 3, n)) / np.sqrt(2 * n)
    Z = (np.transpose(X, (0, 2, 1)) @ X + 0.1 * np.eye(n)).astype(dtype)
    R, info = z.potrf(torch.from_numpy(Z).to("cuda"))
    Ri = z.trtri(R).cpu().numpy().astype(np.float64)
    R = R.cpu().numpy().astype(np.float64)
    u = np.finfo(dtype).eps / 2
    assert info == [0, 0, 0]
    for b in range(3):
        assert np.array_equal(R[b], np.triu(R[b])) and np.array_equal(Ri[b], np.triu(Ri[b]))
        Zb = Z[b].astype(np.float64)
        # Backward errors of the two algorithms: (n + 1) u |R^T||R| and n u |Ri||R||Ri| to first order.
        assert np.all(np.abs(R[b].T @ R[b] - Zb) <= 2 * (n + 8) * u * (np.abs(R[b]).T @ np.abs(R[b])))
        assert np.linalg.norm(R[b] @ Ri[b] - np.eye(n)) <= 4 * (n + 8) * u * np.linalg.norm(R[b]) * np.linalg.norm(Ri[b])


# Diagonal entries whose reciprocal overflows (or is subnormal): an entry of the
# inverse above them is its sum divided by them, 0 or an ordinary number.
@pytest.mark.parametrize("dtype,tiny,small,huge", [("float64", 2.0 ** -1040, 2.0 ** -1050, 2.0 ** 1023),
                                                   ("float32", 2.0 ** -135, 2.0 ** -142, 2.0 ** 127)])
@pytest.mark.parametrize("n", [2, 9, 16])
def test_triangular_inverse_of_extreme_diagonals(z, n, dtype, tiny, small, huge):
    import torch
    R = np.stack([np.eye(n), np.eye(n), np.eye(n)])
    R[0, 0, 0] = tiny                             # nothing above the other columns' ones
    R[1, 0, 0] = tiny
    R[1, 0, 1:] = small
    R[2, 0, 0] = huge
    R[2, 0, 1:] = huge / 4
    Ri = z.trtri(torch.from_numpy(R.astype(dtype)).to("cuda")).cpu().numpy().astype(np.float64)
    top = [1.0 / np.asarray([tiny, tiny, huge], dtype=dtype), [0.0, -small / tiny, -0.25]]
    for b in range(3):
        E = np.eye(n)
        E[0, 0] = top[0][b]
        E[0, 1:] = top[1][b]
        assert np.array_equal(Ri[b], E), b


@pytest.mark.parametrize("at", [0, 15, 16, 40, 63, 64, 99])
def test_cholesky_breakdown_column(z, at):
    import torch
    n = 100
    Z = np.eye(n) * 4.0
    Z[at, at] = -1.0
    if at + 1 < n:
        Z[at + 1, at + 1] = 0.0   # the first bad pivot is the one reported
    R, info = z.potrf(torch.from_numpy(np.stack([Z, np.eye(n)])).to("cuda"))
    assert info == [at + 1, 0]
    assert np.array_equal(R.cpu().numpy()[1], np.eye(n))


def test_cholesky_scaled(z):
    # Pivots from 1e-300 to 1e300: R scales exactly by powers of two.
    import torch
    rng = np.random.default_rng(3)
    X = rng.standard_normal((90, 70))
    Z = X.T @ X
    R0 = z.potrf(torch.from_numpy(Z[None]).to("cuda"))[0].cpu().numpy()[0]
    for e in (-996, -400, 400, 980):
        R = z.potrf(torch.from_numpy(np.ldexp(Z, e)[None]).to("cuda"))[0].cpu().numpy()[0]
        assert np.abs(R - np.ldexp(R0, e // 2)).max() <= 1e-14 * np.ldexp(np.abs(R0).max(), e // 2)


# Every orientation of the pipelined FP64 product at odd extents and at its
# smallest sizes, and the products that stay with the register-staged kernel
# (k < 16, single rows or columns).  Whole numbers: the results are exact.
@pytest.mark.parametrize("m,n,k", [(2, 2, 16), (1, 7, 40), (7, 1, 40), (3, 5, 15), (3, 2, 17), (65, 63, 33),
                                   (64, 64, 64), (129, 131, 100), (191, 65, 129), (63, 257, 257), (130, 258, 1001),
                                   (515, 517, 70), (1031, 1029, 300)])
@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
def test_products_of_whole_numbers(z, m, n, k, ta, tb):
    import torch
    rng = np.random.default_rng(m * n + k)
    A = rng.integers(-9, 10, (2, k, m) if ta else (2, m, k)).astype(np.float64)
    B = rng.integers(-9, 10, (2, n, k) if tb else (2, k, n)).astype(np.float64)
    C = rng.integers(-9, 10, (2, m, n)).astype(np.float64)
    got = z.gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), torch.from_numpy(C).cuda(), transa=ta,
                 transb=tb, alpha=2.0, beta=-3.0).cpu().numpy()
    opa = np.transpose(A, (0, 2, 1)) if ta else A
    opb = np.transpose(B, (0, 2, 1)) if tb else B
    assert np.array_equal(got, 2.0 * (opa @ opb) - 3.0 * C)


@pytest.mark.parametrize("off,lda,ldb,ldc", [(0, 131, 133, 135), (1, 132, 134, 136), (1, 131, 134, 137)])
def test_products_at_odd_offsets(z, off, lda, ldb, ldc):
    # Raw calls: operands that start and step at odd elements.
    import ctypes
    import torch
    rng = np.random.default_rng(off + lda)
    m, n, k, batch = 130, 97, 131, 2
    buf = {c: rng.integers(-9, 10, off + batch * ld * 140 + 1).astype(np.float64) for c, ld in
           (("A", lda), ("B", ldb), ("C", ldc))}
    dv = {c: torch.from_numpy(x).cuda() for c, x in buf.items()}
    ptr = {c: ctypes.c_void_p(t.data_ptr() + 8 * off) for c, t in dv.items()}
    rc = z.lib.zolo_dgemm(z.h, 1, 0, m, n, k, 1.0, ptr["A"], lda, lda * 131 + 1, ptr["B"], ldb, ldb * 97 + 1, 1.0,
                          ptr["C"], ldc, ldc * 97 + 2, batch)
    assert rc == 0
    for b in range(batch):
        a = buf["A"][off + b * (lda * 131 + 1):][:lda * m].reshape(m, lda)[:, :k]
        x = buf["B"][off + b * (ldb * 97 + 1):][:ldb * n].reshape(n, ldb)[:, :k].T
        c = buf["C"][off + b * (ldc * 97 + 2):][:ldc * n].reshape(n, ldc)[:, :m].T
        got = dv["C"].cpu().numpy()[off + b * (ldc * 97 + 2):][:ldc * n].reshape(n, ldc)[:, :m].T
        assert np.array_equal(got, a @ x + c)


@pytest.mark.parametrize("m,n", [(128, 128), (384, 64), (500, 130), (383, 191), (700, 257), (1100, 321)])
@pytest.mark.parametrize("cond", [3.0, 1e6])
def test_steps_of_few_tiles(z, m, n, cond):
    # The products of Cholesky-type (low condition) and QR-type steps in pieces.
    # Stopping bound of the solver 5e-14 for the orthogonality, n eps for H.
    A, U, s, V = W.svd_matrix(m, n, cond, 80 + m, 90 + n)
    Q, H, info = z.pd(dev(A), alpha=1.0, l=0.9 / cond)
    assert info["status"] == 0
    Q, H = Q.cpu().numpy(), H.cpu().numpy()
    assert np.linalg.norm(Q.T @ Q - np.eye(n)) / np.sqrt(n) <= 1e-13
    assert np.linalg.norm(Q @ H - A) / np.linalg.norm(A) <= 1e-13
    assert np.array_equal(H, H.T)
