"""The Cholesky transform's trailing update at the edges of its 16 x 16 blocks, against a 64-bit solve: up to 256 sequences the
advantages are a block column of their own, in memory above their row opens a block row or shares the last one."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [18, 31, 32, 33, 80, 81, 95, 96, 97, 129, 130, 143, 144, 145, 159, 160, 255, 256, 257, 271, 272, 273,
                               287, 288, 400, 401])
def test_trailing_block_edges(gpu_device, m):
    rng = np.random.default_rng(m)
    J = rng.standard_normal((3, m, m + 8))
    K = np.einsum("bij,bkj->bik", J, J).astype(np.float32)
    K = (K + K.transpose(0, 2, 1)) / 2
    A = rng.standard_normal((3, m)).astype(np.float32)
    c, info = isopo.transform(torch.from_numpy(K).to(gpu_device), torch.from_numpy(A).to(gpu_device), "interacting", 0.25)
    c = c.cpu().numpy().astype(np.float64)
    assert info.cpu().tolist() == [0, 0, 0]
    for b in range(3):
        M = K[b].astype(np.float64) + 0.25 * np.eye(m)
        want = np.linalg.solve(M, A[b].astype(np.float64))
        # backward stable in 64 bits (residual below m^2 2^-53 of |M||c|), c rounded to fp32 once
        cond = np.linalg.cond(M)
        assert np.linalg.norm(c[b] - want) <= (2.0 ** -24 + cond * m * m * 2.0 ** -53) * np.linalg.norm(want)
