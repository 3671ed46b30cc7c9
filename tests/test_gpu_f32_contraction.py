"""The fp32 contraction (three bf16 parts per value on the matrix cores) against 64-bit sums, at the edges of its tiles,
token blocks, groups and chunks, and on the values its parts do not cover."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo
from paper_2512_23353_amd import workloads as wl

from helpers import split_plan, to_device

pytestmark = pytest.mark.gpu

# d_in, d_out, lengths, and what they are here for: (tile, groups) per sequence, (tile, groups, chunked) of the sum
SHAPES = [
    (4, 4, [1], (64, 1), (64, 1, False)),
    (64, 64, [16, 0, 15, 17], (64, 1), (64, 1, False)),                      # few short items
    (68, 132, [33, 1, 64], (64, 1), (64, 2, False)),
    (52, 20, [156, 123, 132, 0, 158], (64, 2), (64, 1, True)),
    (128, 260, [700, 31, 0, 1201], (64, 4), (64, 1, True)),                  # few items, long walks: groups
    (580, 916, [18, 10, 43, 54, 24, 59, 59, 0, 43], (128, 1), (64, 2, True)),
    (8, 12, [9000, 0, 17, 21000, 5, 0, 15000], (64, 4), (64, 4, True)),      # more chunks would help
    (36, 1028, [90] * 27, (64, 1), (64, 1, True)),                           # narrow: 64-wide tiles
    (260, 516, list(range(1, 140, 2)), (64, 1), (64, 1, True)),              # more than 64 sequences
    (640, 1284, [150, 90, 1, 47, 0, 128, 300, 16] * 4, (128, 1), (128, 1, True)),  # 128-wide tiles, longest sequence first
]


def _reference(prob, c=None):
    X, D = prob.X.double().numpy(), prob.Delta.double().numpy()
    off = prob.seq_offsets
    G = [D[off[i]:off[i + 1]].T @ X[off[i]:off[i + 1]] for i in range(prob.n_seq)]
    M = [np.abs(D[off[i]:off[i + 1]]).T @ np.abs(X[off[i]:off[i + 1]]) for i in range(prob.n_seq)]
    if c is None:
        return np.stack(G), np.stack(M)
    return sum(ci * g for ci, g in zip(c, G)), sum(abs(ci) * g for ci, g in zip(c, M))


def _bound(n_terms):
    """fp32: every product is right to 2^-23 of itself and every one of at most six sums per sixteen tokens (and one per
    chunk or group, at most 64 + 4) rounds the running sum, itself at most the sum of magnitudes, by 2^-23 at most."""
    return (2 + 6 * -(-n_terms // 16) + 68) * 2.0 ** -23


@pytest.mark.parametrize("case", range(len(SHAPES)))
def test_f32_contraction_edges(gpu_device, case):
    d_in, d_out, lengths, per_sequence, summed = SHAPES[case]
    one, plan = split_plan(d_in, d_out, lengths, True), split_plan(d_in, d_out, lengths, False)
    assert (one.tile, one.groups) == per_sequence and one.longest_first == (d_in == 640)
    assert (plan.tile, plan.groups, plan.n_chunks > 1) == summed
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="f32", seed=400 + case, sigma_delta=1e-2, rho=0.3)
    layer, _ = to_device(prob, gpu_device)
    G, M = _reference(prob)
    stash = torch.full((prob.n_seq, d_out, d_in), float("nan"), device=gpu_device)
    got = isopo.seq_grads(layer, stash).double().cpu().numpy()
    assert (np.abs(got - G) <= _bound(max(lengths)) * M).all()
    c = np.random.default_rng(case).standard_normal(prob.n_seq).astype(np.float32)
    c_dev = torch.from_numpy(c).to(gpu_device)
    for coef, cc in ((c_dev, c), (None, np.ones_like(c))):
        want, mag = _reference(prob, cc.astype(np.float64))
        bound = _bound(sum(lengths) + 16 * len(lengths)) * mag
        dW = isopo.weighted_grad(layer, coef).double().cpu().numpy()
        assert (np.abs(dW - want) <= bound).all()
        old = torch.ones((d_out, d_in), device=gpu_device)
        dW = isopo.weighted_grad(layer, coef, None, 0.5, old).double().cpu().numpy()
        assert (np.abs(dW - want - 0.5) <= bound + 2.0 ** -23 * (64 + 4) * (0.5 + mag)).all()


@pytest.mark.parametrize("dims", [(64, 96), (640, 1284)])
@pytest.mark.parametrize("what", ["tiny", "huge", "inf", "nan"])
def test_f32_contraction_outside_the_parts_range(gpu_device, dims, what):
    """Values whose bf16 parts would be subnormal or infinite: as exact as ever, and infinities and NaN stay in the
    rows and columns they belong to."""
    d_in, d_out = dims
    prob = wl.custom_layer(d_in, d_out, [40, 90, 3, 17] * 4, dtype="f32", seed=77, sigma_delta=1.0)
    X, D = prob.X, prob.Delta
    if what == "tiny":
        D *= 2.0 ** -112
    elif what == "huge":
        X *= 2.0 ** -20
        D[45, 3] = 3.4e38                                  # rounds to infinity in bf16
    else:
        D[45, 3] = float(what)
    layer, _ = to_device(prob, gpu_device)
    with np.errstate(all="ignore"):
        G, M = _reference(prob)
    got = isopo.seq_grads(layer).double().cpu().numpy()
    if what in ("tiny", "huge"):
        # the plain fp32 form rounds once per two tokens; 2^-149: the products' own underflow
        assert (np.abs(got - G) <= (2 + 90) * 2.0 ** -23 * M + 90 * 2.0 ** -149).all()
        return
    fin = np.isfinite(G)
    assert not fin[1, 3].any() and fin.sum() == fin.size - d_in
    assert np.array_equal(np.isnan(got), np.isnan(G)) and np.array_equal(np.isinf(got), np.isinf(G))
    assert (np.abs(got[fin] - G[fin]) <= (2 + 90) * 2.0 ** -23 * M[fin]).all()


@pytest.mark.parametrize("dims", [(64, 96), (640, 1284), (128, 260)])
@pytest.mark.parametrize("what", ["row", "column", "against large", "subnormal", "coefficient", "products"])
def test_f32_contraction_small_operands(gpu_device, dims, what):
    """Operands below 2^-110, where fp32 carries more bits than three bf16 parts can, whose products are of ordinary size
    or stand beside ordinary ones: each output as exact as ever."""
    d_in, d_out = dims
    lengths = [40, 90, 3, 17] if dims == (128, 260) else [40, 90, 3, 17] * 4
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="f32", seed=78, sigma_delta=1.0)
    X, D = prob.X, prob.Delta
    c = np.random.default_rng(5).uniform(0.5, 2.0, prob.n_seq).astype(np.float32)
    if what == "row":
        D[:, 5] *= 2.0 ** -122
    elif what == "column":
        X[:, 7] *= 2.0 ** -122
    elif what == "against large":
        D *= 2.0 ** -122
        X *= 2.0 ** 60
    elif what == "subnormal":
        D *= 2.0 ** -138
        X *= 2.0 ** 90
    elif what == "coefficient":
        c *= np.float32(2.0 ** -122)
        X *= 2.0 ** 60
    else:                                                  # ordinary operands, products down to where fp32 ends
        D *= 2.0 ** -80
        X *= 2.0 ** -62
    layer, _ = to_device(prob, gpu_device)
    G, M = _reference(prob)
    got = isopo.seq_grads(layer).double().cpu().numpy()
    # 2^-149: sums below fp32's normal range
    assert (np.abs(got - G) <= (2 + 90) * 2.0 ** -23 * M + 90 * 2.0 ** -149).all()
    # c times a subnormal Delta is rounded to 2^-149 before it is multiplied
    want, mag = _reference(prob, c.astype(np.float64))
    lost = 2.0 ** -149 * (prob.X.double().abs().sum(0).numpy()[None, :] + 6 * len(lengths) * 90)
    dW = isopo.weighted_grad(layer, torch.from_numpy(c).to(gpu_device)).double().cpu().numpy()
    assert (np.abs(dW - want) <= _bound(sum(lengths) + 16 * len(lengths)) * mag + lost).all()


@pytest.mark.parametrize("dims", [(64, 96), (640, 1284)])
def test_f32_contraction_of_one_and_two_tokens(gpu_device, dims):
    """One token: every product rounded once.  Two: each product and the sum rounded once at most, 2^-24 each."""
    lengths = [1, 2, 0, 1, 40, 2] * 4
    prob = wl.custom_layer(*dims, lengths, dtype="f32", seed=79, sigma_delta=1.0)
    layer, _ = to_device(prob, gpu_device)
    G, M = _reference(prob)
    got = isopo.seq_grads(layer).double().cpu().numpy()
    for i, n in enumerate(lengths):
        if n <= 2:
            assert (np.abs(got[i] - G[i]) <= n * 2.0 ** -24 * M[i]).all(), i
    one = wl.custom_layer(*dims, [1, 0], dtype="f32", seed=80, sigma_delta=1.0)
    layer, _ = to_device(one, gpu_device)
    c = np.array([0.7, 3.0], dtype=np.float32)
    for coef, cc, roundings in ((None, np.ones(2), 1), (torch.from_numpy(c).to(gpu_device), c.astype(np.float64), 2)):
        want, mag = _reference(one, cc)
        dW = isopo.weighted_grad(layer, coef).double().cpu().numpy()
        assert (np.abs(dW - want) <= roundings * 2.0 ** -24 * (1 + 2.0 ** -23) * mag).all()
