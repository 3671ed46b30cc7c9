"""The one-pass Gram kernel of 129 to 256 sequences against 64-bit products: every number of 32-row blocks, stashes shorter
than a slice, of a slice and a bit, and of several slices per workgroup with a short last one."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [129, 159, 160, 161, 191, 192, 193, 223, 224, 225, 255, 256])
def test_row_blocks(gpu_device, m):
    gen = torch.Generator(device=gpu_device).manual_seed(m)
    for n in (8, 128, 136, 32768 + 56, 128 * 256 * 3 + 8):
        S = (torch.randn((m, n), generator=gen, device=gpu_device) + 0.3).to(torch.bfloat16)
        K = isopo.stash_gram(S).cpu().numpy()
        S = S.double().cpu().numpy()
        assert np.array_equal(K, K.T), n
        # products exact to 2^-23; a workgroup's sums of sixteen, one after the other, then 16 slots and 16 waves
        chain = 16 + (n // 128 // 256 + 1) * 8 + 32 + 2
        assert (np.abs(K - S @ S.T) <= chain * 2.0 ** -23 * (np.abs(S) @ np.abs(S).T)).all(), n
