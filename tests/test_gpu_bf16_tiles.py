"""The bf16 contraction against 64-bit sums where the output tile or the kind of store changes: row-major stashes on both
sides of each line."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo
from paper_2512_23353_amd import workloads as wl

from helpers import to_device

pytestmark = pytest.mark.gpu


def _sums(prob):
    """Per-sequence gradients in 64 bits and the same sums of magnitudes."""
    X, D = prob.X.double().numpy(), prob.Delta.double().numpy()
    off = prob.seq_offsets
    rows = [slice(off[i], off[i + 1]) for i in range(prob.n_seq)]
    return (np.stack([D[r].T @ X[r] for r in rows]), np.stack([np.abs(D[r]).T @ np.abs(X[r]) for r in rows]))


@pytest.mark.parametrize("d_in,d_out,lens", [
    (264, 1280, [300, 256, 511, 0, 260, 400]),   # long on average: non-temporal
    (264, 1280, [300, 31, 0, 33, 200, 1]),       # short: through the L2
    (8, 136, [256] * 3), (8, 136, [255] * 3),    # the line itself
    (520, 1288, [20, 0, 40] * 6),                # wide tiles, ragged both ways
])
def test_row_major_stash_stores(gpu_device, d_in, d_out, lens):
    prob = wl.custom_layer(d_in, d_out, lens, dtype="bf16", seed=d_out, sigma_delta=1e-2, rho=0.3)
    layer, _ = to_device(prob, gpu_device)
    G, M = _sums(prob)
    S = isopo.seq_grads(layer, torch.full(G.shape, float("nan"), dtype=torch.bfloat16, device=gpu_device))
    # exact products, at most one rounding of the running sum per token (2^-23 truncated), one rounding to bf16
    bound = 2.0 ** -8 * np.abs(G) + max(lens) * 2.0 ** -23 * 1.01 * M
    assert (np.abs(S.double().cpu().numpy() - G) <= bound).all()
