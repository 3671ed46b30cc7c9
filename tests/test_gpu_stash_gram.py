"""The streaming Gram kernels against 64-bit products: every number of 16- and 32-row blocks, stashes shorter than one
stage and with a short last stage, and a small workspace whose output rows are formed and reduced in chunks."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo
from paper_2512_23353_amd import workloads as wl

from helpers import to_device

pytestmark = pytest.mark.gpu


def _check(K, S, what):
    S = S.double().cpu().numpy().reshape(S.shape[0], -1)
    want = S @ S.T
    K = K.cpu().numpy()
    assert np.array_equal(K, K.T), what
    # products exact to 2^-23 and sums to sqrt-free worst case: chains of 64 (fp32) or n_elem/1024/16 matrix-core sums of a
    # workgroup's wave, four waves and the flushes, then 64 bits and one rounding; against the sum of magnitudes
    n = S.shape[1]
    chain = 64 + 4 + n // (256 * 64) + 2
    bound = chain * 2.0 ** -23 * (np.abs(S) @ np.abs(S).T)
    assert (np.abs(K - want) <= bound).all(), what


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m", [1, 2, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113, 128])
def test_stash_gram_row_blocks(gpu_device, dtype, m):
    gen = torch.Generator(device=gpu_device).manual_seed(m)
    for n in (8, 56, 2056, 40968):
        S = (torch.randn((m, n), generator=gen, device=gpu_device) + 0.3).to(dtype)
        _check(isopo.stash_gram(S), S, f"{dtype} m={m} n={n}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m", [5, 40, 100])
def test_layer_gram_in_chunks_of_rows(gpu_device, dtype, m):
    """ws_min: 256 output rows at a time, the last chunk shorter than the one that set the number of slots."""
    prob = wl.custom_layer(64, 776, [9] * m, dtype=dtype, seed=m, sigma_delta=1e-2, rho=0.3)
    layer, _ = to_device(prob, gpu_device)
    K, _ = isopo.layer_gram(layer, "materialised")
    _, _, small = isopo.gram_plan(layer, "materialised")
    K2, _ = isopo.layer_gram(layer, "materialised", workspace=isopo.alloc_workspace(small, gpu_device))
    stash = isopo.seq_grads(layer)
    _check(K2, stash, "chunks")
    # the same products, summed in another order
    scale = torch.sqrt(K.diagonal()[:, None] * K.diagonal()[None, :])
    assert float(((K - K2).abs() / scale).max()) <= 2.0 ** -23 * 140
