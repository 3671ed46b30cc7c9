"""The norms of a Gram matrix, a wave per row, where rows end within a wave's loads and workgroups within the rows."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 3, 5, 63, 64, 65, 128, 257])
def test_gram_norms_rows(gpu_device, m):
    K = np.random.default_rng(m).standard_normal((m, m)).astype(np.float32)
    f2, g2 = isopo.gram_norms(torch.from_numpy(K).to(gpu_device))
    want = (K.astype(np.float64) ** 2).mean(axis=1)
    assert (np.abs(f2.cpu().numpy() - want) <= 2.0 ** -23 * want).all()
    assert np.array_equal(g2.cpu().numpy(), np.diag(K))
