"""The Cholesky transform with the matrix in registers at the edges of its 16 x 16 blocks and of what its launches take, with NaN in
the upper triangle, which is not read, against a 64-bit solve."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 15, 16, 17, 31, 33, 48, 63, 64, 65, 79, 81, 112, 127, 128, 129, 177, 240, 241, 255, 256])
def test_registers(gpu_device, m):
    rng = np.random.default_rng(m)
    J = rng.standard_normal((3, m, m + 8))
    K = np.einsum("bij,bkj->bik", J, J).astype(np.float32)
    K = np.tril(K) + np.tril(K, -1).transpose(0, 2, 1)
    A = rng.standard_normal((3, m)).astype(np.float32)
    upper = np.where(np.triu(np.ones((m, m), bool), 1), np.float32("nan"), K)
    c, info = isopo.transform(torch.from_numpy(upper).to(gpu_device), torch.from_numpy(A).to(gpu_device), "interacting", 0.01,
                              isopo.REG_REL_TRACE)
    c = c.cpu().numpy().astype(np.float64)
    assert info.cpu().tolist() == [0, 0, 0]
    for b in range(3):
        M = K[b].astype(np.float64)
        M += 0.01 * np.trace(M) / m * np.eye(m)
        want = np.linalg.solve(M, A[b].astype(np.float64))
        # backward stable in 64 bits (residual below m^2 2^-53 of |M||c|; a lambda of 0.01 is an fp32 value away), c rounded once
        cond = np.linalg.cond(M)
        assert np.linalg.norm(c[b] - want) <= (2.0 ** -24 + 2.0 ** -24 + cond * m * m * 2.0 ** -53) * np.linalg.norm(want)


@pytest.mark.parametrize("m", [1, 8, 9, 16, 63, 65, 96, 97, 130, 1021])
def test_fisher_rows(gpu_device, m):
    rng = np.random.default_rng(m)
    K = rng.standard_normal((2, m, m)).astype(np.float32)
    A = rng.standard_normal((2, m)).astype(np.float32)
    c, _ = isopo.transform(torch.from_numpy(K).to(gpu_device), torch.from_numpy(A).to(gpu_device), "fisher", 0.5, isopo.REG_REL_TRACE)
    f2 = (K.astype(np.float64) ** 2).mean(axis=2)
    want = A / np.sqrt(f2 + 0.5 * f2.mean(axis=1, keepdims=True))
    # 64-bit sums of positive terms, one rounding to fp32
    assert (np.abs(c.cpu().numpy() - want) <= 2.0 ** -23 * np.abs(want)).all()


@pytest.mark.parametrize("m", [8, 9, 48, 49, 64, 65, 104, 105])
@pytest.mark.parametrize("batch", [257, 513])
def test_fisher_batches(gpu_device, m, batch):
    """More problems than compute units: fewer waves for each of the smaller ones."""
    rng = np.random.default_rng(m)
    K = rng.standard_normal((batch, m, m)).astype(np.float32)
    A = rng.standard_normal((batch, m)).astype(np.float32)
    c, info = isopo.transform(torch.from_numpy(K).to(gpu_device), torch.from_numpy(A).to(gpu_device), "fisher", 0.5, isopo.REG_REL_TRACE)
    f2 = (K.astype(np.float64) ** 2).mean(axis=2)
    want = A / np.sqrt(f2 + 0.5 * f2.mean(axis=1, keepdims=True))
    # as above
    assert (np.abs(c.cpu().numpy() - want) <= 2.0 ** -23 * np.abs(want)).all() and not info.any()
