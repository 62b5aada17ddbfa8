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
