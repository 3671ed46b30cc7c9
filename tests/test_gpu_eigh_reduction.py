"""The tridiagonal reduction at the sizes where its sixteen-wide groups of columns, its rows per lane and the last two
columns meet: eigenvalues and reconstruction to rounding, with columns that are already reduced among them."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [4, 8, 14, 15, 16, 18, 30, 32, 34, 46, 47, 48, 50, 62, 64, 66, 96, 112, 126, 128])
def test_reduction_sizes(gpu_device, m):
    rng = np.random.default_rng(m)
    J = rng.standard_normal((m, 2 * m))
    gram = J @ J.T
    split = gram.copy()                                   # two blocks that do not meet: a column is through early
    split[: m // 2, m // 2:] = split[m // 2:, : m // 2] = 0.0
    K = np.stack([gram, split, np.diag(np.arange(1.0, m + 1))]).astype(np.float32)
    D, U, info = isopo.ntk_eigh(torch.from_numpy(K).to(gpu_device))
    assert info.tolist() == [0] * len(K)
    D, U = D.cpu().numpy(), U.cpu().numpy()
    # backward stable: a modest multiple of n rounding errors of the norm
    tol = 16 * (m + 8) * 2.0 ** -53
    for b in range(len(K)):
        Kd = K[b].astype(np.float64)
        Kd = (Kd + Kd.T) / 2
        ref = np.linalg.eigvalsh(Kd)
        size = np.abs(ref).max()
        assert np.abs(D[b] - ref).max() <= tol * size
        assert np.abs(U[b].T @ U[b] - np.eye(m)).max() <= tol
        assert np.abs((U[b] * D[b]) @ U[b].T - Kd).max() <= tol * size
