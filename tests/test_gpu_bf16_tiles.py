"""The bf16 contraction against 64-bit sums where the output tile or the kind of store changes: row-major stashes and
weighted sums on both sides of each line."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo
from paper_2512_23353_amd import workloads as wl

from helpers import bf16_plan, to_device, walk_plan

pytestmark = pytest.mark.gpu


def _sums(prob):
    """Per-sequence gradients in 64 bits and the same sums of magnitudes."""
    X, D = prob.X.double().numpy(), prob.Delta.double().numpy()
    off = prob.seq_offsets
    rows = [slice(off[i], off[i + 1]) for i in range(prob.n_seq)]
    return (np.stack([D[r].T @ X[r] for r in rows]), np.stack([np.abs(D[r]).T @ np.abs(X[r]) for r in rows]))


@pytest.mark.parametrize("d_in,d_out,lens", [
    (264, 1280, [300, 256, 511, 0, 260, 400]),   # long on average
    (264, 1280, [300, 31, 0, 33, 200, 1]),       # short
    (8, 136, [256] * 3), (8, 136, [255] * 3),    # one narrow tile
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


@pytest.mark.parametrize("d_in,d_out,lens,tile", [
    (264, 1280, [70] * 100, 128), (256, 1280, [70] * 100, 256),     # a ragged width, and none: tile order needs wide tiles
    (520, 1288, [25] * 20, 128), (1000, 2728, [420] * 24, 256),     # either side of the modelled line
])
def test_row_major_tile(gpu_device, d_in, d_out, lens, tile):
    prob = wl.custom_layer(d_in, d_out, lens, dtype="bf16", seed=d_in, sigma_delta=1e-2, rho=0.3)
    layer, _ = to_device(prob, gpu_device)
    assert isopo.contraction_plan(layer.ref(), True)["tile"] == tile
    S = isopo.seq_grads(layer)
    for i in (0, 7, len(lens) - 1):
        r = slice(int(prob.seq_offsets[i]), int(prob.seq_offsets[i + 1]))
        X, D = layer.X[r].double(), layer.Delta[r].double()
        G, M = D.T.contiguous() @ X, D.abs().T.contiguous() @ X.abs()
        assert ((S[i].double() - G).abs() <= 2.0 ** -8 * G.abs() + lens[i] * 2.0 ** -23 * 1.01 * M).all(), i


@pytest.mark.parametrize("d_in,d_out,lens,tile", [
    (512, 1288, [2500, 1, 0, 33, 5000, 4100] * 2, 128),      # 12 wide tiles in chunks: narrow ones in fewer
    (1536, 1536, [900, 31, 64] * 11, 128),                   # 36
    (1024, 2816, [16500], 128), (256, 4352, [16500], 256),   # one sequence, either side of what the last-level cache takes
    (1536, 2560, [7000, 0, 12001, 2500], 256),               # past it as well
])
def test_weighted_sum_in_chunks(gpu_device, d_in, d_out, lens, tile):
    plan = bf16_plan(d_in, d_out, lens, False, weighted=True)
    assert plan.tile == tile and plan.n_chunks > 1 and bf16_plan(d_in, d_out, lens, False).tile == 256
    prob = wl.custom_layer(d_in, d_out, lens, dtype="bf16", seed=d_out, sigma_delta=1e-2, rho=0.3)
    layer, _ = to_device(prob, gpu_device)
    c = torch.randn(len(lens), generator=torch.Generator().manual_seed(3))
    if len(lens) > 1:
        c[1] = 0.0
    got = isopo.weighted_grad(layer, c.to(gpu_device))
    w = torch.repeat_interleave(c, torch.tensor(lens)).to(gpu_device).double()[:, None]
    X, D = layer.X.double(), layer.Delta.double() * w
    G, M = D.T.contiguous() @ X, D.abs().T.contiguous() @ X.abs()
    # exact products; one rounding of the running sum per token, three per change of sequence and one per chunk
    bound = (sum(lens) + 3 * len(lens) + 64) * 2.0 ** -23 * M
    assert ((got.double() - G).abs() <= bound).all()


@pytest.mark.parametrize("d_in,d_out,lens,budget", [
    (264, 1280, [260] * 100, 64), (520, 1288, [300] * 60, 8), (1032, 2048, [780, 0, 801, 333] * 2, 224), (1032, 2048, [780] * 8, 256)])
def test_budget_on_ragged_widths(gpu_device, d_in, d_out, lens, budget):
    """Row-major layers that take 128-wide tiles without a budget: the launch's plan keeps the budget all the same, and the
    stash is the unlimited call's bit for bit.  (The scratch words are cleared by a launch on a budget and by no other: that
    shows that a budget reached the kernel, not its size, which is the plan's.)"""
    prob = wl.custom_layer(d_in, d_out, lens, dtype="bf16", seed=d_in, sigma_delta=1e-2, rho=0.3)
    layer, _ = to_device(prob, gpu_device)
    assert isopo.contraction_plan(layer.ref(), True)["tile"] == 128
    assert bf16_plan(d_in, d_out, lens, True, budget=True).tile == 256
    assert 8 * walk_plan(d_in, d_out, lens, budget)[0].per_xcd <= budget
    want = isopo.seq_grads(layer)
    for kw in ({}, {"layout": isopo.STASH_ROW_MAJOR}):
        queue = torch.full((8,), 12345, dtype=torch.int32, device=gpu_device)
        got = isopo.seq_grads(layer, torch.full_like(want, float("nan")), max_workgroups=budget, queue=queue, **kw)
        assert (queue != 12345).all()
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
