"""Odd extents, leading dimensions and offsets in the pipelined FP64 GEMM
(dgemm_pipe_kernel in csrc/gemm.hip), replayed on the CPU with real values:
the chunk addresses, the clamp of edge rows, the mended pair of an odd edge,
the shifted ragged slice and the zeroing, against the operand itself.  Every
load must lie inside the operand's storage."""

import numpy as np
import pytest

BK = 16


def coords(R, kc):
    slot = np.arange(R * BK // 2)
    if not kc:
        kk = slot // (R // 2)
        return 2 * ((slot % (R // 2)) ^ ((kk & 1) * 8)), kk
    r = slot // (BK // 2)
    return r, 2 * ((slot % (BK // 2)) ^ (r & 7))


def slice_values(mem, R, kc, ext, ld, lo0, kb, ke, t, tri):
    """The R x 16 block that slice t of a tile stores (rows lo0.., k from kb + 16 t)."""
    r, kk = coords(R, kc)
    last = ext - 1 if kc else ext - 2
    g = np.maximum(np.minimum(lo0 + r, last), 0)
    kq = kb + BK * t
    k0 = min(kq, ke - BK)
    off = kk + g * ld if kc else g + kk * ld
    off = off + k0 * (1 if kc else ld)
    assert off.min() >= 0 and off.max() + 1 < mem.size
    v = np.stack([mem[off], mem[off + 1]])
    if not kc and ext % 2 == 1 and lo0 + R > ext:   # the pair of the last row
        v[0] = np.where(lo0 + r == ext - 1, v[1], v[0])
    out = np.full((R, 2 * BK), np.nan)
    for h in (0, 1):
        rr, gk = r + (0 if kc else h), k0 + kk + (h if kc else 0)
        ok = (gk >= kq) & (gk < ke) & tri(lo0 + rr, gk)
        out[rr, gk - k0 + (k0 - kq) + BK] = np.where(ok, v[h], 0.0)
    return kq - BK, out   # column c of out is k = kq - BK + c


@pytest.mark.parametrize("kc", [False, True])
@pytest.mark.parametrize("R,ext,k,pad,tri", [
    (64, 2, 16, 0, None), (64, 3, 17, 0, None), (64, 63, 31, 1, None), (64, 65, 129, 0, None),
    (128, 129, 40, 3, None), (128, 191, 33, 0, None), (64, 131, 131, 0, "upper"), (64, 131, 131, 2, "lower"),
    (128, 1, 20, 0, None)])
def test_odd_edges(kc, R, ext, k, pad, tri):
    if not kc and ext < 2:
        pytest.skip("a single row along the pairs goes to gemm_kernel")
    rng = np.random.default_rng(R + ext + k)
    X = rng.standard_normal((ext, k)) + 3.0          # op(A): rows, k
    ld = (k if kc else ext) + pad
    mem = np.full((ext - 1) * ld + k if kc else (k - 1) * ld + ext, np.nan)
    idx = np.arange(k)[None, :] + np.arange(ext)[:, None] * ld if kc else \
        np.arange(ext)[:, None] + np.arange(k)[None, :] * ld
    mem[idx] = X
    inside = {None: lambda i, q: np.ones_like(q, bool), "upper": lambda i, q: q >= i,
              "lower": lambda i, q: q <= i}[tri]
    want = np.where(inside(*np.indices((ext, k))), X, 0.0)
    for lo0 in range(0, ext, R):
        kb = lo0 if tri == "upper" else 0
        ke = min(k, lo0 + R) if tri == "lower" else k
        got = np.zeros((R, k))
        for t in range(-(-(ke - kb) // BK)):
            k_at, blk = slice_values(mem, R, kc, ext, ld, lo0, kb, ke, t, inside)
            for c in range(2 * BK):
                if not np.isnan(blk[: min(R, ext - lo0), c]).all() and 0 <= k_at + c < k:
                    got[:, k_at + c] += np.where(np.isnan(blk[:, c]), 0.0, blk[:, c])
        rows = min(R, ext - lo0)
        assert np.array_equal(got[:rows, kb:ke], want[lo0:lo0 + rows, kb:ke])
