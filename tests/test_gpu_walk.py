"""The bf16 contractions whose workgroups walk lists of (sequence, tile) pairs, against 64-bit sums where the lists and the walks
over the tokens change: tile counts that are no multiple of eight, sequences that are empty or shorter than the loads run ahead,
more of them than are sorted by length, sums of more tiles than compute units on either side of the first token block."""
import pytest
import torch

from paper_2512_23353_amd import isopo
from paper_2512_23353_amd import workloads as wl

from helpers import bf16_plan, to_device, walk_plan

pytestmark = pytest.mark.gpu


def _layer(d_in, d_out, lens, device):
    return to_device(wl.custom_layer(d_in, d_out, lens, dtype="bf16", seed=len(lens) + d_in, sigma_delta=1e-2, rho=0.3), device)[0]


def _check_stash(layer, S, lens):
    for i, n in enumerate(lens):
        r = slice(int(layer.off_host[i]), int(layer.off_host[i + 1]))
        X, D = layer.X[r].double(), layer.Delta[r].double()
        G, M = D.T.contiguous() @ X, D.abs().T.contiguous() @ X.abs()
        # exact products, at most one rounding of the running sum per token (2^-23 truncated), one rounding to bf16
        assert ((S[i].double() - G).abs() <= 2.0 ** -8 * G.abs() + n * 2.0 ** -23 * 1.01 * M).all(), i


@pytest.mark.parametrize("d_in,d_out,lens,tile", [
    (264, 776, [0, 1, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160] * 4, 128),  # every length of walk there is to get wrong
    (264, 2056, [40, 0, 7, 300, 1, 97] * 7, 128),                            # 51 tiles, 42 sequences
    (1000, 2728, [900, 33, 600] * 5, 256),                                   # 44 wide tiles
    (4104, 4360, [800, 0, 33, 700], 256),                                    # 306, few sequences
    (8, 136, [3, 0, 40] * 100, 128),                                         # more sequences than are sorted
])
def test_row_major_lists(gpu_device, d_in, d_out, lens, tile):
    assert bf16_plan(d_in, d_out, lens, True).tile == tile
    layer = _layer(d_in, d_out, lens, gpu_device)
    S = torch.full((len(lens), d_out, d_in), float("nan"), dtype=torch.bfloat16, device=gpu_device)
    _check_stash(layer, isopo.seq_grads(layer, S), lens)


@pytest.mark.parametrize("d_in,d_out,lens", [
    (256, 768, [0, 1, 31, 32, 33, 64, 65, 96, 97, 128, 129] * 9), (768, 2816, [40, 0, 200, 33, 1, 640, 97] * 2),
    (256, 512, [3, 0, 40] * 100)])
def test_tile_order_lists(gpu_device, d_in, d_out, lens):
    """The same elements as in the row-major stash, bit for bit, so the two layouts' weighted sums are equal."""
    layer = _layer(d_in, d_out, lens, gpu_device)
    layout, tile = isopo.stash_layout(layer)
    assert layout == isopo.STASH_TILE_ORDER
    rows = isopo.seq_grads(layer)
    _check_stash(layer, rows, lens)
    tiled = isopo.seq_grads(layer, torch.full_like(rows, float("nan")), layout=layout)
    c = torch.randn(len(lens), generator=torch.Generator().manual_seed(1)).to(gpu_device)
    assert torch.equal(isopo.weighted_grad(layer, c, rows), isopo.weighted_grad(layer, c, tiled, layout=layout))


@pytest.mark.parametrize("lens,beta", [([1], 0.0), ([32, 33], 0.5), ([0, 200, 64, 0, 1, 31], 0.0), ([97] * 5, -1.5), ([0, 40], 2.0)])
@pytest.mark.parametrize("weighted", [True, False])
def test_sums_of_many_tiles(gpu_device, lens, beta, weighted):
    d_in, d_out = 4104, 4368                     # 17 x 18 wide tiles, ragged both ways
    plan = bf16_plan(d_in, d_out, lens, False, weighted=weighted)
    assert plan.tile == 256 and plan.n_chunks == 1 and plan.tiles_m * plan.tiles_n > 256
    layer = _layer(d_in, d_out, lens, gpu_device)
    gen = torch.Generator().manual_seed(len(lens))
    c = torch.randn(len(lens), generator=gen)
    if len(lens) != 2 or lens[0] == 0:           # [0, 40]: no sequence is left
        c[1:2] = 0.0
    start = torch.randn((d_out, d_in), generator=gen).to(gpu_device)
    got = isopo.weighted_grad(layer, c.to(gpu_device) if weighted else None, beta=beta, dW=start.clone())
    w = torch.repeat_interleave(c, torch.tensor(lens)).to(gpu_device).double()[:, None] if weighted else 1.0
    X, D = layer.X.double(), layer.Delta.double() * w
    G = beta * start.double() + D.T.contiguous() @ X
    M = abs(beta) * start.double().abs() + D.abs().T.contiguous() @ X.abs()
    # exact products; one rounding of the running sum per token, three per change of sequence, three of the result
    assert ((got.double() - G).abs() <= (sum(lens) + 3 * len(lens) + 3) * 2.0 ** -23 * M).all()


@pytest.mark.parametrize("lens,beta", [([2048], 0.0), ([1000, 0, 33, 1100], 0.5), ([31] * 70, 0.0)])
@pytest.mark.parametrize("weighted", [True, False])
def test_uncut_sums_of_one_round(gpu_device, lens, beta, weighted):
    d_in, d_out = 3000, 5000                     # 240 wide tiles, ragged both ways: one to a workgroup
    plan = bf16_plan(d_in, d_out, lens, False, weighted=weighted)
    assert plan.tile == 256 and plan.n_chunks == 1 and plan.tiles_m * plan.tiles_n <= 256
    layer = _layer(d_in, d_out, lens, gpu_device)
    gen = torch.Generator().manual_seed(len(lens))
    c = torch.randn(len(lens), generator=gen)
    start = torch.randn((d_out, d_in), generator=gen).to(gpu_device)
    got = isopo.weighted_grad(layer, c.to(gpu_device) if weighted else None, beta=beta, dW=start.clone())
    w = torch.repeat_interleave(c, torch.tensor(lens)).to(gpu_device).double()[:, None] if weighted else 1.0
    X, D = layer.X.double(), layer.Delta.double() * w
    G = beta * start.double() + D.T.contiguous() @ X
    M = abs(beta) * start.double().abs() + D.abs().T.contiguous() @ X.abs()
    # as above
    assert ((got.double() - G).abs() <= (sum(lens) + 3 * len(lens) + 3) * 2.0 ** -23 * M).all()


@pytest.mark.parametrize("d_in,d_out,lens,budget,kind", [
    (1000, 2728, [8000] + [100] * 31, 0, "alone"), (1000, 2728, [100] * 20 + [8000] + [31] * 11, 128, "alone"),
    (520, 1288, [20] * 399 + [9000], 0, "alone"),                    # more sequences than a byte counts
    (768, 264, [2230, 0, 4000, 33] * 7, 0, "single"), (264, 264, [1, 0, 40], 0, "single"),
    (768, 1024, [900] + [300, 0, 1, 33] * 99, 0, "ranges"), (768, 392, [2230, 0, 4000, 33] * 7, 0, "alone"),
    (512, 512, [3000] + [60, 0] * 60, 0, "alone"),
])
def test_arrangements(gpu_device, d_in, d_out, lens, budget, kind):
    """Launches whose pairs are dealt out in other ways: long pairs whose workgroups take no other, a workgroup per pair, ranges of
    the list; in either layout, and twice in a row into the same stash."""
    plan, _ = walk_plan(d_in, d_out, lens, budget)
    assert kind == ("alone" if any(plan.alone) else ("dealt", "ranges", "single")[plan.kind])
    layer = _layer(d_in, d_out, lens, gpu_device)
    layout = isopo.stash_layout(layer)[0]
    queue = torch.zeros(8, dtype=torch.int32, device=gpu_device)
    S = torch.full((len(lens), d_out, d_in), float("nan"), dtype=torch.bfloat16, device=gpu_device)
    for _ in range(2):
        S.fill_(float("nan"))
        _check_stash(layer, isopo.seq_grads(layer, S, max_workgroups=budget, queue=queue if budget else None), lens)
    if layout == isopo.STASH_TILE_ORDER:
        tiled = isopo.seq_grads(layer, torch.full_like(S, float("nan")), layout=layout)
        c = torch.randn(len(lens), generator=torch.Generator().manual_seed(1)).to(gpu_device)
        assert torch.equal(isopo.weighted_grad(layer, c, S), isopo.weighted_grad(layer, c, tiled, layout=layout))


@pytest.mark.parametrize("d_in,d_out,lens,tile,rows,columns,kind", [
    (1000, 1032, [90, 0, 400, 64] * 5, 128, 9, 8, "dealt"), (1032, 1288, [33, 500, 0] * 4, 128, 11, 9, "dealt"),
    (1160, 1032, [90, 0, 400, 64] * 5, 128, 9, 10, "dealt"), (1288, 1288, [33, 500, 0] * 4, 128, 11, 11, "dealt"),
    (1000, 264, [20] * 200, 128, 3, 8, "ranges"), (1160, 264, [20] * 200, 128, 3, 10, "ranges"),
    (1160, 1288, [40, 7], 128, 11, 10, "single"), (1160, 1032, [2000, 3] * 3, 128, 9, 10, "alone"),
    (1024, 512, [90, 0, 400, 64] * 5, 128, 4, 8, "alone"), (1280, 512, [2000, 3] * 3, 128, 4, 10, "single"),       # tile order
    (2304, 768, [33, 500, 0] * 4, 256, 3, 9, "alone"), (2560, 1024, [33, 500, 0] * 8, 256, 4, 10, "dealt"),
    (2048, 2048, [90, 0, 400, 64] * 9, 256, 8, 8, "dealt"), (1792, 5632, [40, 200] * 2, 256, 22, 7, "dealt"),
    (2560, 2568, [90, 0, 400, 64] * 9, 256, 11, 10, "dealt"), (2600, 2568, [90, 0, 400, 64] * 9, 256, 11, 11, "dealt"),      # row by row
    (1792, 5888, [40, 200] * 2, 256, 23, 7, "dealt"), (2312, 4104, [300, 33, 700] * 4, 256, 17, 10, "dealt"),    # 161 tiles and more
    (1800, 2568, [300, 33, 700] * 4, 128, 21, 15, "dealt"), (2312, 1032, [90, 0, 400, 64] * 5, 128, 9, 19, "dealt")])
def test_narrow_strips(gpu_device, d_in, d_out, lens, tile, rows, columns, kind):
    """Tiles in strips of four columns (launches of up to 160 tiles), the last of one to four, on both tiles, in either layout and
    every way of dealing the pairs out; and launches of more tiles, in strips of eight."""
    plan, (walk, _) = bf16_plan(d_in, d_out, lens, True), walk_plan(d_in, d_out, lens)
    assert (plan.tile, plan.tiles_m, plan.tiles_n) == (tile, rows, columns)
    assert kind == ("alone" if any(walk.alone) else ("dealt", "ranges", "single")[walk.kind])
    layer = _layer(d_in, d_out, lens, gpu_device)
    layout, _ = isopo.stash_layout(layer)
    rows = isopo.seq_grads(layer, torch.full((len(lens), d_out, d_in), float("nan"), dtype=torch.bfloat16, device=gpu_device))
    _check_stash(layer, rows, lens)
    if layout == isopo.STASH_TILE_ORDER:
        tiled = isopo.seq_grads(layer, torch.full_like(rows, float("nan")), layout=layout)
        c = torch.randn(len(lens), generator=torch.Generator().manual_seed(1)).to(gpu_device)
        assert torch.equal(isopo.weighted_grad(layer, c, rows), isopo.weighted_grad(layer, c, tiled, layout=layout))
