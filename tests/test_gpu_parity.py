"""Parity of the HIP path (through the C ABI) with the CPU fp64 oracle.

Every comparison is element by element on the same seeded input bytes.
Tolerances are the benchmark definition's: 1e-4 relative for fp32 inputs, 2e-2
relative for bf16 inputs with fp32 accumulation (norm-wise, with element
guards; see helpers.py).
"""
import numpy as np
import pytest
import torch

from oracle import isopo_oracle as orc
from paper_2512_23353_amd import isopo
from paper_2512_23353_amd import workloads as wl

from helpers import TOL, assert_K_close, assert_c_close, assert_dW_close, oracle_step, rel_err, to_device, walk_plan

pytestmark = pytest.mark.gpu


def _check_step(prob, device, path, variant, lam, reg_mode=0, chunk_rows=None):
    tol = TOL[prob.dtype]
    layer, A = to_device(prob, device)
    out = isopo.layer_step(layer, A, variant, lam, reg_mode, path)
    torch.cuda.synchronize()
    ref = oracle_step(prob, variant, lam, reg_mode, chunk_rows)
    what = f"{prob.name}/{path}/{variant}"
    assert out["path"] == path or path == "auto"
    assert int(out["info"].item()) == ref["info"] == 0
    assert_K_close(out["K"].cpu().numpy(), ref["K"], tol, what)
    assert_c_close(out["c"].cpu().numpy(), ref["c"], tol, what)
    assert_dW_close(out["dW"].cpu().numpy(), ref["dW"], tol, what, ref["dW_abs"])
    # the same coefficients contracted again from X and Delta (no stash)
    dW2 = isopo.weighted_grad(layer, out["c"])
    assert_dW_close(dW2.cpu().numpy(), ref["dW"], tol, what + "/recompute", ref["dW_abs"])
    return out, ref


@pytest.mark.parametrize("path", ["materialised", "ghost"])
@pytest.mark.parametrize("variant", ["fisher", "interacting"])
@pytest.mark.parametrize("reg", [(1e-3, isopo.REG_ABSOLUTE), (1e-3, isopo.REG_REL_TRACE)])
def test_config1_fp32(gpu_device, path, variant, reg):
    w = wl.CONFIGS["config1"]
    prob = wl.make_layer(w, w.projections[0])
    _check_step(prob, gpu_device, path, variant, reg[0], reg[1])


@pytest.mark.parametrize("path", ["materialised", "ghost"])
def test_config1_correlated(gpu_device, path):
    """Rollouts of one prompt correlate: off-diagonal K is a sizeable fraction
    of the diagonal, so the interacting solve really mixes sequences."""
    w = wl.CONFIGS["config1"]
    prob = wl.make_layer(w, w.projections[0], rho=1.0)
    out, ref = _check_step(prob, gpu_device, path, "interacting", 0.05, isopo.REG_REL_TRACE)
    K = ref["K"]
    offd = np.abs(K - np.diag(np.diag(K))).max() / np.diag(K).mean()
    assert offd > 0.1


EDGE_CASES = [
    ("ragged", 256, 384, [100, 37, 1, 0, 250, 64]),
    ("all_single_tokens", 64, 128, [1] * 40),
    ("one_huge_many_tiny", 128, 256, [3, 1, 700, 2, 5, 1, 1, 9]),
    ("one_sequence", 256, 128, [333]),
    ("narrow_dims", 72, 200, [31, 32, 33, 65]),
    ("empty_first_and_last", 128, 128, [0, 50, 0, 0, 70, 0]),
    # 11 token tiles of 128: the bf16 ghost launch walks its tile pairs in two bands of tile rows, and its
    # grid is padded to whole runs per XCD
    ("eleven_token_tiles", 72, 136, [400, 3, 520, 1, 377]),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", EDGE_CASES, ids=[c[0] for c in EDGE_CASES])
@pytest.mark.parametrize("path", ["materialised", "ghost"])
def test_ragged_edge_cases(gpu_device, dtype, case, path):
    _, d_in, d_out, lengths = case
    prob = wl.custom_layer(d_in, d_out, lengths, dtype=dtype, seed=11, sigma_delta=1e-2)
    _check_step(prob, gpu_device, path, "interacting", 1e-2, isopo.REG_REL_TRACE)
    _check_step(prob, gpu_device, path, "fisher", 1e-2, isopo.REG_REL_TRACE)


def _tile_order_index(d_out, d_in, T):
    """Row-major element index of every position of a stash in tile order (the layout include/isopo.h
    documents for ISOPO_STASH_TILE_ORDER), written out from that description."""
    idx = np.empty(d_out * d_in, dtype=np.int64)
    pos = 0
    l = np.arange(64)
    q = np.arange(8)
    for tm in range(d_out // T):
        for tn in range(d_in // T):
            for quad in range(4):
                r0, c0 = tm * T + (quad >> 1) * (T // 2), tn * T + (quad & 1) * (T // 2)
                for strip in range(T // 32):
                    for piece in range(T // 64):
                        rows = r0 + strip * 16 + 4 * (l[:, None] // 16) + q[None, :] % 4
                        cols = c0 + piece * 32 + l[:, None] % 16 + 16 * (q[None, :] // 4)
                        idx[pos:pos + 512] = (rows * d_in + cols).reshape(-1)
                        pos += 512
    assert pos == d_out * d_in
    return idx


TILE_ORDER_CASES = [
    # name, d_in, d_out, lengths: 256x256 tiles with the persistent launch (6 tiles x 48 sequences), 128x128 tiles
    ("tile256_persistent", 768, 512, [int(x) for x in np.random.default_rng(3).integers(0, 90, 48)]),
    ("tile128", 256, 512, [70, 0, 129, 33, 300]),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("path", ["materialised", "ghost"])
def test_layer_without_tokens(gpu_device, dtype, path):
    """The empty input: every sequence has length zero (X and Delta have no rows, their device pointers may be
    null).  K = 0 and dW = beta dW exactly; with an absolute regulariser both variants have coefficients
    (A / lambda, A / sqrt(lambda)); with the relative one reg = 0: the Fisher variant gives c = 0, the interacting
    one reports the failing pivot.  One shape whose bf16 stash is kept in tile order, one that is row-major only."""
    for d_in, d_out in ((256, 512), (72, 200)):
        prob = wl.custom_layer(d_in, d_out, [0, 0, 0, 0, 0], dtype=dtype, seed=3)
        for variant in ("interacting", "fisher"):
            out, ref = _check_step(prob, gpu_device, path, variant, 0.5, isopo.REG_ABSOLUTE)
            assert not out["K"].any() and not out["dW"].any()
            assert np.abs(ref["c"]).min() > 0.1
        layer, A = to_device(prob, gpu_device)
        out = isopo.layer_step(layer, A, "fisher", 0.5, isopo.REG_REL_TRACE, path)
        assert int(out["info"].item()) == 0 and not out["c"].any() and not out["dW"].any()
        out = isopo.layer_step(layer, A, "interacting", 0.5, isopo.REG_REL_TRACE, path)
        assert int(out["info"].item()) == 1 and bool(torch.isnan(out["c"]).all())
        # the contractions from X and Delta alone: beta dW, bit for bit
        dW0 = torch.randn((d_out, d_in), device=gpu_device)
        for c in (None, torch.ones(prob.n_seq, device=gpu_device)):
            dW = dW0.clone()
            isopo.weighted_grad(layer, c, None, 0.5, dW)
            assert torch.equal(dW, 0.5 * dW0)
            dW = torch.full_like(dW0, float("nan"))
            isopo.weighted_grad(layer, c, None, 0.0, dW)
            assert not dW.any()


@pytest.mark.parametrize("case", TILE_ORDER_CASES, ids=[c[0] for c in TILE_ORDER_CASES])
def test_stash_in_tile_order(gpu_device, case):
    """A bf16 layer whose dimensions are multiples of 256 keeps its stash in the matrix cores' own order.
    The elements are the row-major stash's at the documented positions (to one bf16 rounding: the two
    kernels use MFMAs of different depth, so their fp32 sums may differ in the last bit before the
    rounding); K, c and dW of the whole step match the oracle; the stash-weighted sum gives the same bits
    from either layout of one stash."""
    name, d_in, d_out, lengths = case
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=29, sigma_delta=1e-2, rho=0.4)
    layer, A = to_device(prob, gpu_device)
    layout, T = isopo.stash_layout(layer)
    assert layout == isopo.STASH_TILE_ORDER and T == (256 if name.startswith("tile256") else 128)
    plan = isopo.contraction_plan(layer.ref(), True)
    assert plan["tile"] == T
    row_major = isopo.seq_grads(layer)
    tiled = isopo.seq_grads(layer, layout=isopo.STASH_TILE_ORDER)
    budget = isopo.seq_grads(layer, layout=isopo.STASH_TILE_ORDER, max_workgroups=256)
    torch.cuda.synchronize()
    idx = _tile_order_index(d_out, d_in, T)
    rm = row_major.view(torch.int16).cpu().numpy().reshape(prob.n_seq, -1)
    rm_f = row_major.float().cpu().numpy().reshape(prob.n_seq, -1)[:, idx]
    tl = tiled.view(torch.int16).cpu().numpy().reshape(prob.n_seq, -1)
    assert np.array_equal(budget.view(torch.int16).cpu().numpy().reshape(prob.n_seq, -1), tl)   # same kernel, other launch
    tl_f = tiled.float().cpu().numpy().reshape(prob.n_seq, -1)
    assert np.all(np.abs(tl_f - rm_f) <= 2.0 ** -7 * np.abs(rm_f) + 1e-30)
    assert np.mean(tl == rm[:, idx]) > 0.99
    # the whole step through the kept stash
    _check_step(prob, gpu_device, "materialised", "interacting", 1e-2, isopo.REG_REL_TRACE)
    K_fast, ws = isopo.layer_gram(layer, "materialised", keep_stash=isopo.KEEP_FAST)
    K_rm, ws_rm = isopo.layer_gram(layer, "materialised", keep_stash=isopo.KEEP_ROW_MAJOR)
    torch.cuda.synchronize()
    n = prob.n_seq * d_out * d_in
    assert np.array_equal(ws[: 2 * n].view(torch.int16).cpu().numpy().reshape(prob.n_seq, -1), tl)
    assert np.array_equal(ws_rm[: 2 * n].view(torch.int16).cpu().numpy().reshape(prob.n_seq, -1), rm)
    assert rel_err(K_fast.cpu().numpy(), K_rm.cpu().numpy()) < 1e-5
    c = torch.from_numpy(np.random.default_rng(4).standard_normal(prob.n_seq).astype(np.float32)).to(gpu_device)
    dW0 = torch.from_numpy(np.random.default_rng(5).standard_normal((d_out, d_in)).astype(np.float32)).to(gpu_device)
    # one stash in both layouts: the tile-order one, and its elements put back in row-major order
    inv = np.empty_like(idx)
    inv[idx] = np.arange(idx.size)
    back = torch.from_numpy(tl[:, inv].copy()).to(gpu_device).view(torch.bfloat16).view(prob.n_seq, d_out, d_in)
    for beta in (0.0, 0.5):
        a = isopo.weighted_grad(layer, c, ws, beta, dW0.clone(), layout=isopo.STASH_TILE_ORDER)
        b = isopo.weighted_grad(layer, c, back, beta, dW0.clone())
        torch.cuda.synchronize()
        assert torch.equal(a, b), f"beta={beta}"
    # a row-major stash through the same entry point
    assert torch.equal(isopo.weighted_grad(layer, c, ws_rm, layout=isopo.STASH_ROW_MAJOR), isopo.weighted_grad(layer, c, ws_rm))


@pytest.mark.parametrize("case", TILE_ORDER_CASES[:2] + [("row_major_264x512", 264, 512, [40, 3, 0, 77, 130])],
                         ids=lambda c: c[0])
def test_weighted_grad_from_stash_into_bf16(gpu_device, case):
    """dW in bf16 (`mod.grad +=` on a bf16 parameter): with beta = 0 the bits are the fp32 result's, rounded to
    nearest even; with beta != 0 the old bf16 values enter in fp32 before the one rounding; the oracle's dW is met
    within the bf16 tolerance.  Both layouts of the stash."""
    name, d_in, d_out, lengths = case
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=31, sigma_delta=1e-2, rho=0.3)
    layer, A = to_device(prob, gpu_device)
    layout, _ = isopo.stash_layout(layer)
    assert layout == (isopo.STASH_ROW_MAJOR if name.startswith("row_major") else isopo.STASH_TILE_ORDER)
    K, ws = isopo.layer_gram(layer, "materialised", keep_stash=isopo.KEEP_FAST)
    c, info = isopo.transform(K, A, "interacting", 1e-2, isopo.REG_REL_TRACE)
    full = isopo.weighted_grad(layer, c, ws, layout=layout)
    half = isopo.weighted_grad_stash_bf16(layer, c, ws, layout)
    torch.cuda.synchronize()
    assert half.dtype == torch.bfloat16 and torch.equal(half, full.to(torch.bfloat16))
    ref = oracle_step(prob, "interacting", 1e-2, isopo.REG_REL_TRACE)
    assert_dW_close(half.float().cpu().numpy(), ref["dW"], TOL["bf16"], f"{name} bf16 dW", ref["dW_abs"])
    # accumulation into an existing bf16 gradient
    old = torch.from_numpy(np.random.default_rng(6).standard_normal((d_out, d_in)).astype(np.float32)).to(gpu_device)
    old = (old * full.abs().mean()).to(torch.bfloat16)
    for beta in (1.0, 0.5):
        got = isopo.weighted_grad_stash_bf16(layer, c, ws, layout, beta, old.clone())
        want = isopo.weighted_grad(layer, c, ws, beta, old.float(), layout=layout).to(torch.bfloat16)
        torch.cuda.synchronize()
        assert torch.equal(got, want), f"beta={beta}"
    # fp32 layers have no bf16 gradient
    prob32 = wl.custom_layer(64, 128, [5, 9], dtype="f32", seed=32)
    layer32, _ = to_device(prob32, gpu_device)
    stash32 = isopo.seq_grads(layer32)
    with pytest.raises(isopo.IsopoError) as e:
        isopo.weighted_grad_stash_bf16(layer32, torch.ones(2, device=gpu_device), stash32, isopo.STASH_ROW_MAJOR, 0.0,
                                       torch.zeros((128, 64), dtype=torch.bfloat16, device=gpu_device))
    assert e.value.status == 3


def test_stash_layout_falls_back_to_row_major(gpu_device):
    """Dimensions that are not multiples of 256, or fp32 inputs: keep_stash = 2 leaves the row-major stash,
    and asking for tile order is refused."""
    for dtype, d_in, d_out in (("bf16", 264, 512), ("f32", 256, 256)):
        prob = wl.custom_layer(d_in, d_out, [40, 3, 77], dtype=dtype, seed=30, sigma_delta=1e-2)
        layer, _ = to_device(prob, gpu_device)
        assert isopo.stash_layout(layer) == (isopo.STASH_ROW_MAJOR, 0)
        _, ws = isopo.layer_gram(layer, "materialised", keep_stash=isopo.KEEP_FAST)
        ref = isopo.seq_grads(layer)
        torch.cuda.synchronize()
        nbytes = ref.numel() * ref.element_size()
        assert torch.equal(ws[:nbytes], ref.view(torch.uint8).reshape(-1))
        c = torch.ones(prob.n_seq, device=gpu_device)
        for call in (lambda: isopo.seq_grads(layer, layout=isopo.STASH_TILE_ORDER),
                     lambda: isopo.weighted_grad(layer, c, ws, layout=isopo.STASH_TILE_ORDER)):
            with pytest.raises(isopo.IsopoError) as e:
                call()
            assert e.value.status == 3


GHOST_SPLIT_CASES = [
    # name, d_in, d_out, lengths: wide layers on few tokens, where the bf16 ghost launch cuts the features
    # into ranges; 64-feature tails, and an operand with fewer 64-feature slices than ranges
    ("two_ranges_feature_tails", 1096, 1000, [100, 37, 1, 0, 250, 64]),
    ("three_ranges_narrow_delta", 3000, 40, [31, 32, 33, 65]),
    ("eight_ranges_one_tile", 4096, 4096, [50, 9, 60]),
    ("three_tile_pairs", 2048, 1536, [130, 1, 70, 20]),
]


@pytest.mark.parametrize("case", GHOST_SPLIT_CASES, ids=[c[0] for c in GHOST_SPLIT_CASES])
def test_ghost_feature_ranges(gpu_device, case):
    _, d_in, d_out, lengths = case
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=23, sigma_delta=1e-2, rho=0.5)
    layer, _ = to_device(prob, gpu_device)
    n_tiles = (sum(lengths) + 127) // 128
    # the workspace carries the fp32 parts (two 128x128 products) of every (tile pair, range): at least two ranges
    _, full, _ = isopo.gram_plan(layer, "ghost")
    assert full >= n_tiles * (n_tiles + 1) // 2 * 2 * (2 * 128 * 128 * 4)
    _check_step(prob, gpu_device, "ghost", "interacting", 1e-2, isopo.REG_REL_TRACE)
    Kg, _ = isopo.layer_gram(layer, "ghost")
    Km, _ = isopo.layer_gram(layer, "materialised")
    torch.cuda.synchronize()
    assert torch.equal(Kg, Kg.T)
    assert rel_err(Km.cpu().numpy(), Kg.cpu().numpy()) < 1e-3


GHOST_LONG_CASES = [
    # microbatches long enough for more tile pairs than resident workgroups (several rounds, XCD runs): whole
    # tiles; a ragged last tile with a feature count that is no multiple of 64; many short sequences whose
    # boundaries cross the 32 x 32 blocks, empty ones among them; one long sequence against short ones
    ("whole_tiles", 256, 384, [512] * 8),
    ("ragged_end_odd_features", 264, 200, [700, 3, 1500, 0, 1100, 801]),
    ("many_short_sequences", 128, 256, [37, 5, 90, 0, 1, 64, 33, 150] * 10 + [1000]),
    ("one_long_sequence", 512, 128, [4000, 60, 60, 120]),
]


@pytest.mark.parametrize("case", GHOST_LONG_CASES, ids=[c[0] for c in GHOST_LONG_CASES])
def test_ghost_long_microbatches(gpu_device, case):
    """The ghost form on 4000 tokens and more (hundreds of 128 x 128 token-pair tiles, no feature ranges): K
    against the oracle in full, bit-symmetric, and equal to the materialised path's within rounding."""
    _, d_in, d_out, lengths = case
    assert sum(lengths) >= 4000
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=29, sigma_delta=1e-2, rho=0.5)
    layer, _ = to_device(prob, gpu_device)
    Kg, _ = isopo.layer_gram(layer, "ghost")
    Km, _ = isopo.layer_gram(layer, "materialised")
    torch.cuda.synchronize()
    K_ref = orc.layer_ntk(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets, chunk_rows=64,
                          matrix_product=True)
    assert_K_close(Kg.cpu().numpy(), K_ref, TOL["bf16"], f"ghost long {case[0]}")
    assert torch.equal(Kg, Kg.T)
    assert rel_err(Km.cpu().numpy(), Kg.cpu().numpy()) < 1e-3
    empty = [i for i, n in enumerate(lengths) if n == 0]
    assert all(not Kg[i].any() for i in empty)


def test_both_gram_paths_agree_and_are_symmetric(gpu_device):
    prob = wl.custom_layer(512, 768, [300, 517, 33, 260, 128], dtype="bf16", seed=4, sigma_delta=1e-2, rho=0.7)
    layer, _ = to_device(prob, gpu_device)
    Km, _ = isopo.layer_gram(layer, "materialised")
    Kg, _ = isopo.layer_gram(layer, "ghost")
    Km2, _ = isopo.layer_gram(layer, "materialised")
    torch.cuda.synchronize()
    assert torch.equal(Km, Km.T) and torch.equal(Kg, Kg.T)
    assert torch.equal(Km, Km2), "materialised K must be bit-reproducible"
    assert rel_err(Km.cpu().numpy(), Kg.cpu().numpy()) < 1e-3


def test_chunked_workspace_matches_whole(gpu_device):
    """With only the minimum workspace the stash is formed and reduced in chunks
    of output rows; K must not change beyond summation order."""
    prob = wl.custom_layer(256, 1024, [200, 77, 300, 150], dtype="bf16", seed=5, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    _, full, mn = isopo.gram_plan(layer, "materialised")
    assert mn < full
    K_whole, _ = isopo.layer_gram(layer, "materialised")
    ws = isopo.alloc_workspace(mn, gpu_device)
    K_chunk, _ = isopo.layer_gram(layer, "materialised", workspace=ws)
    torch.cuda.synchronize()
    ref = orc.layer_ntk(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets)
    assert_K_close(K_chunk.cpu().numpy(), ref, TOL["bf16"], "chunked")
    assert rel_err(K_chunk.cpu().numpy(), K_whole.cpu().numpy()) < 1e-5
    with pytest.raises(isopo.IsopoError) as e:
        isopo.layer_gram(layer, "materialised", workspace=isopo.alloc_workspace(mn - 4096, gpu_device))
    assert e.value.status == 4
    with pytest.raises(isopo.IsopoError) as e:
        isopo.layer_gram(layer, "materialised", workspace=ws, keep_stash=True)
    assert e.value.status == 4


def test_stash_holds_per_sequence_gradients(gpu_device):
    prob = wl.custom_layer(128, 256, [90, 10, 45], dtype="f32", seed=6, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    _, ws = isopo.layer_gram(layer, "materialised", keep_stash=True)
    torch.cuda.synchronize()
    stash = ws[: 3 * 256 * 128 * 4].view(torch.float32).reshape(3, 256, 128).cpu().numpy()
    G = orc.seq_logprob_grads(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets)
    assert rel_err(stash, G) < 1e-5


@pytest.mark.parametrize("dims,n_seq", [((768, 512), 48), ((1536, 256), 44), ((768, 512), 3)])
def test_per_sequence_gradients_with_xcd_work_ranges(gpu_device, dims, n_seq):
    """Tile counts that are no multiple of eight (6 tiles of 256x256, or 24/12 of
    128x128 with few sequences): the XCDs have uneven numbers of (sequence, tile)
    pairs, dealt out or in ranges as the launch's plan says.  Ragged lengths with
    empty sequences; every per-sequence gradient in the stash and K are checked, so
    a pair that no workgroup took cannot pass."""
    d_in, d_out = dims
    rng = np.random.default_rng(77)
    lengths = [int(x) for x in rng.integers(0, 160, n_seq)]
    lengths[1] = 0
    lengths[-1] = 0
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=12, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    plan = isopo.contraction_plan(layer.ref(), True)
    assert plan["tiles"] % 8 != 0 or n_seq == 3
    K, ws = isopo.layer_gram(layer, "materialised", keep_stash=True)
    torch.cuda.synchronize()
    stash = ws[: n_seq * d_out * d_in * 2].view(torch.bfloat16).reshape(n_seq, d_out, d_in).float().cpu().numpy()
    G = orc.seq_logprob_grads(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets)
    for i in range(n_seq):
        if lengths[i] == 0:
            assert not stash[i].any()
        else:
            assert rel_err(stash[i], G[i]) < 4e-3, i        # one bf16 rounding of an fp32 sum
    assert_K_close(K.cpu().numpy(), orc.ntk_from_seq_grads(G), TOL["bf16"], f"xcd ranges {dims} B={n_seq}")


@pytest.mark.parametrize("from_stash", [True, False])
def test_weighted_grad_accumulates_with_beta(gpu_device, from_stash):
    prob = wl.custom_layer(256, 256, [100, 64, 90], dtype="bf16", seed=7, sigma_delta=1e-2)
    layer, A = to_device(prob, gpu_device)
    _, ws = isopo.layer_gram(layer, "materialised", keep_stash=True)
    dW0 = torch.randn(256, 256, device=gpu_device) * 1e-2
    dW = dW0.clone()
    isopo.weighted_grad(layer, A, ws if from_stash else None, beta=0.5, dW=dW)
    torch.cuda.synchronize()
    G = orc.seq_logprob_grads(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets)
    ref = orc.weighted_grad(G, prob.A, dW0.cpu().numpy(), 0.5)
    assert_dW_close(dW.cpu().numpy(), ref, TOL["bf16"], "beta")


def test_reinforce_baseline_is_weighted_grad_with_advantages(gpu_device):
    prob = wl.custom_layer(384, 512, [257, 100, 511, 64], dtype="bf16", seed=8, sigma_delta=1e-2)
    layer, A = to_device(prob, gpu_device)
    dW = isopo.weighted_grad(layer, A)
    torch.cuda.synchronize()
    ref = oracle_step(prob, "fisher", 0.0)["dW_reinforce"]
    assert_dW_close(dW.cpu().numpy(), ref, TOL["bf16"], "reinforce")


def _random_gram(rng, m, rank_extra=8, scale=1.0):
    J = rng.standard_normal((m, m + rank_extra)) * scale
    J += 0.5 * scale * rng.standard_normal((1, m + rank_extra))    # common component -> dense K
    return (J @ J.T).astype(np.float32)


@pytest.mark.parametrize("m", [1, 2, 4, 7, 8, 9, 15, 16, 17, 31, 32, 33, 48, 49, 64, 96, 97, 128, 129, 200, 256, 300, 512, 513, 1024])
@pytest.mark.parametrize("variant", ["fisher", "interacting"])
def test_transform_sizes(gpu_device, m, variant):
    rng = np.random.default_rng(100 + m)
    batch = 3
    K = np.stack([_random_gram(rng, m, scale=1.0 + b) for b in range(batch)])
    A = rng.standard_normal((batch, m)).astype(np.float32)
    for lam, mode in [(1e-2, isopo.REG_REL_TRACE), (0.5, isopo.REG_ABSOLUTE)]:
        c, info = isopo.transform(torch.from_numpy(K).to(gpu_device), torch.from_numpy(A).to(gpu_device),
                                  variant, lam, mode)
        torch.cuda.synchronize()
        assert info.cpu().tolist() == [0] * batch
        for b in range(batch):
            if variant == "fisher":
                ref = orc.coeff_fisher(K[b], A[b], lam, mode)
            else:
                ref, oinfo = orc.coeff_interacting(K[b], A[b], lam, mode)
                assert oinfo == 0
            # K enters as given fp32 bits on both sides; the solve itself runs in fp64
            assert_c_close(c[b].cpu().numpy(), ref, 1e-5, f"transform m={m} {variant}")


def test_transform_reports_not_positive_definite(gpu_device):
    K = np.array([[4.0, 2.0, 0.0], [2.0, 1.0, 0.0], [0.0, 0.0, 1.0]], dtype=np.float32)
    Kb = np.stack([K, np.eye(3, dtype=np.float32), -np.eye(3, dtype=np.float32)])
    A = np.ones((3, 3), dtype=np.float32)
    c, info = isopo.transform(torch.from_numpy(Kb).to(gpu_device), torch.from_numpy(A).to(gpu_device),
                              "interacting", 0.0)
    torch.cuda.synchronize()
    assert info.cpu().tolist() == [2, 0, 1]
    assert [orc.coeff_interacting(Kb[b], A[b], 0.0)[1] for b in range(3)] == [2, 0, 1]
    c = c.cpu().numpy()
    assert np.all(np.isnan(c[0])) and np.all(np.isnan(c[2])) and np.allclose(c[1], 1.0)
    # with a regulariser the singular problem is solvable and unique
    c, info = isopo.transform(torch.from_numpy(K).to(gpu_device), torch.from_numpy(A[0]).to(gpu_device),
                              "interacting", 0.1)
    ref, _ = orc.coeff_interacting(K, A[0], 0.1)
    assert info.item() == 0
    assert_c_close(c.cpu().numpy(), ref, 1e-5, "regularised singular")
    # fisher: an all-zero row with reg 0 gives c_i = 0
    Kz = np.diag([1.0, 0.0, 2.0]).astype(np.float32)
    c, info = isopo.transform(torch.from_numpy(Kz).to(gpu_device), torch.from_numpy(A[0]).to(gpu_device), "fisher", 0.0)
    assert c.cpu().numpy()[1] == 0.0 and np.all(np.isfinite(c.cpu().numpy()))


@pytest.mark.parametrize("m,k", [(64, 16), (64, 17), (64, 40), (128, 128), (200, 32), (200, 33), (200, 150), (200, 200),
                                 (600, 17), (600, 600), (1024, 1009)])
def test_transform_failing_pivot_in_any_panel(gpu_device, m, k):
    """The k-th pivot is exactly -1 (row and column k - 1 of a dense positive definite matrix are cleared, the
    diagonal entry set to -1): info = k and a NaN fill, wherever k falls in the panels of the factorisation;
    the other problem of the batch is solved."""
    rng = np.random.default_rng(1000 * m + k)
    good = _random_gram(rng, m)
    bad = good.copy()
    bad[k - 1, :] = 0.0
    bad[:, k - 1] = 0.0
    bad[k - 1, k - 1] = -1.0
    K = np.stack([bad, good])
    A = rng.standard_normal((2, m)).astype(np.float32)
    c, info = isopo.transform(torch.from_numpy(K).to(gpu_device), torch.from_numpy(A).to(gpu_device), "interacting",
                              1e-3, isopo.REG_ABSOLUTE)
    torch.cuda.synchronize()
    assert info.cpu().tolist() == [k, 0]
    assert orc.coeff_interacting(bad, A[0], 1e-3, isopo.REG_ABSOLUTE)[1] == k
    c = c.cpu().numpy()
    assert np.all(np.isnan(c[0]))
    ref, oinfo = orc.coeff_interacting(good, A[1], 1e-3, isopo.REG_ABSOLUTE)
    assert oinfo == 0
    assert_c_close(c[1], ref, 1e-5, f"m={m}, the solvable problem beside a failing one")


def test_schedule_probes(gpu_device):
    """The two diagnostics behind the benchmark's schedule probe: the eight-wave contraction gives the four-wave
    launch's dW, which is isopo_weighted_grad's (to fp32 rounding: with few tiles the token range is split and the
    parts are added with atomics); the LDS-DMA probe runs for every wave count and ring depth and rejects what it
    does not serve."""
    # enough tokens for the plan to take the 256x256 tile (with a token split), ragged tile edges in d_out
    prob = wl.custom_layer(1024, 1100 // 8 * 8, [3000, 0, 777, 1, 6500, 3100], dtype="bf16", seed=41, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    assert isopo.contraction_plan(layer.ref(), False)["tile"] == 256
    want = isopo.weighted_grad(layer, None)
    four = isopo.probe_contraction_waves(layer, 4)
    eight = isopo.probe_contraction_waves(layer, 8)
    torch.cuda.synchronize()
    for got in (four, eight):
        assert float((got - want).norm() / want.norm()) < 1e-6
    G = orc.seq_logprob_grads(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets)
    ones = np.ones(prob.n_seq)
    assert_dW_close(eight.cpu().numpy(), orc.weighted_grad(G, ones), TOL["bf16"], "eight waves", orc.weighted_grad_abs(G, ones))
    small = wl.custom_layer(64, 128, [40, 9], dtype="bf16", seed=42)
    small_layer, _ = to_device(small, gpu_device)
    with pytest.raises(isopo.IsopoError) as e:
        isopo.probe_contraction_waves(small_layer, 8)
    assert e.value.status == 3
    with pytest.raises(isopo.IsopoError) as e:
        isopo.probe_contraction_waves(layer, 6)
    assert e.value.status == 1
    buf = torch.ones(8 * 32768 * 4, dtype=torch.uint8, device=gpu_device)
    sink = torch.zeros(64, dtype=torch.float32, device=gpu_device)
    for waves in (2, 4, 8, 16):
        for stages in (2, 4):
            isopo.probe_lds_dma(buf, waves, stages, 16, 50, sink)
    torch.cuda.synchronize()
    for bad in (dict(waves=3), dict(stages=3), dict(workgroups=0), dict(iters=0)):
        kw = dict(waves=4, stages=2, workgroups=8, iters=10)
        kw.update(bad)
        with pytest.raises(isopo.IsopoError) as e:
            isopo.probe_lds_dma(buf, kw["waves"], kw["stages"], kw["workgroups"], kw["iters"], sink)
        assert e.value.status == 1
    with pytest.raises(isopo.IsopoError):
        isopo.probe_lds_dma(buf[:1000], 4, 2, 8, 10, sink)


def test_bad_arguments_on_device_calls(gpu_device):
    prob = wl.custom_layer(128, 128, [10, 20], dtype="bf16", seed=9)
    layer, A = to_device(prob, gpu_device)
    with pytest.raises(isopo.IsopoError) as e:
        isopo.layer_gram(layer, "ghost", keep_stash=True)
    assert e.value.status == 1
    with pytest.raises(isopo.IsopoError) as e:
        isopo.transform(torch.eye(4, device=gpu_device), torch.ones(4, device=gpu_device), "interacting", -1.0)
    assert e.value.status == 1
    K = torch.eye(200, device=gpu_device)
    with pytest.raises(isopo.IsopoError) as e:
        isopo.transform(K, torch.ones(200, device=gpu_device), "interacting", 0.1,
                        workspace=isopo.alloc_workspace(1024, gpu_device))
    assert e.value.status == 4


@pytest.mark.parametrize("n_seq", [129, 200, 256, 300])
def test_more_than_128_sequences(gpu_device, n_seq):
    """Large batches take the super-block Gram kernel on the materialised path
    (and the global-scratch Cholesky in the transform); both Gram paths and the
    whole step are compared with the oracle."""
    rng = np.random.default_rng(n_seq)
    lengths = rng.integers(1, 40, size=n_seq)
    lengths[5] = 0
    prob = wl.custom_layer(136, 264, lengths, dtype="bf16", seed=n_seq, sigma_delta=1e-2, rho=0.3)
    layer, A = to_device(prob, gpu_device)
    ref = oracle_step(prob, "interacting", 1e-2, isopo.REG_REL_TRACE)
    for path in ("materialised", "ghost"):
        out = isopo.layer_step(layer, A, "interacting", 1e-2, isopo.REG_REL_TRACE, path)
        torch.cuda.synchronize()
        what = f"n_seq={n_seq}/{path}"
        assert int(out["info"].item()) == 0
        assert_K_close(out["K"].cpu().numpy(), ref["K"], TOL["bf16"], what)
        assert_c_close(out["c"].cpu().numpy(), ref["c"], TOL["bf16"], what)
        assert_dW_close(out["dW"].cpu().numpy(), ref["dW"], TOL["bf16"], what, ref["dW_abs"])
    # chunked accumulation over output rows with the minimum workspace
    _, full, mn = isopo.gram_plan(layer, "materialised")
    K_chunk, _ = isopo.layer_gram(layer, "materialised", workspace=isopo.alloc_workspace(mn, gpu_device))
    torch.cuda.synchronize()
    assert_K_close(K_chunk.cpu().numpy(), ref["K"], TOL["bf16"], f"n_seq={n_seq}/chunked")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dims", [(256, 640), (640, 256)])
def test_prescaled_weighted_grad(gpu_device, dtype, dims):
    """Scaling the narrower operand's rows by c_tok and contracting unweighted
    equals the weighted contraction; the scaled rows themselves are the exact
    product rounded once to the storage type."""
    d_in, d_out = dims
    prob = wl.custom_layer(d_in, d_out, [70, 0, 129, 33, 300], dtype=dtype, seed=21, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    rng = np.random.default_rng(5)
    c = rng.standard_normal(prob.n_seq).astype(np.float32)
    c_dev = torch.from_numpy(c).to(gpu_device)
    dW = isopo.weighted_grad_prescaled(layer, c_dev)
    scaled = isopo.scale_rows(layer.X, layer, c_dev)
    torch.cuda.synchronize()
    G = orc.seq_logprob_grads(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets)
    assert_dW_close(dW.cpu().numpy(), orc.weighted_grad(G, c), TOL[dtype], "prescaled", orc.weighted_grad_abs(G, c))
    c_tok = np.repeat(c.astype(np.float64), np.diff(prob.seq_offsets))
    exact = orc.widen(wl.to_oracle(prob.X)) * c_tok[:, None]
    got = orc.widen(wl.to_oracle(scaled))
    ulp = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -23
    assert np.all(np.abs(got - exact) <= ulp * np.abs(exact) + 1e-300)


WEIGHTED_CASES = [
    # d_in, d_out, lengths: whole 256x256 tiles then a split tail; token split on both tile sizes (a dozen or
    # more chunks whose boundaries fall inside sequences); one tile, no split; many short sequences
    (4096, 4200, [700, 1, 0, 900, 447]),
    (256, 384, [3000, 1400, 1, 4200, 333, 4100]),
    (512, 256, [3000, 1400, 1, 4200, 333, 4100]),
    (200, 136, [3000, 1400, 1, 4200, 333, 4100]),
    (1024, 768, [31, 32, 33, 0, 64, 65, 1, 2, 500, 95, 97]),
    (768, 512, [5] * 70 + [0, 0, 129] + [1] * 40),
    # the library's limit of 1024 sequences, most of them one or two tokens long, some empty: a boundary in nearly
    # every token block; and 300 sequences on a layer that takes the token split
    (512, 256, [int(x) for x in np.random.default_rng(1).integers(0, 6, 1024)]),
    (256, 256, [int(x) for x in np.random.default_rng(2).integers(0, 90, 300)]),
]


@pytest.mark.parametrize("case", range(len(WEIGHTED_CASES)))
@pytest.mark.parametrize("beta", [0.0, 0.75])
def test_weighted_contraction_from_x_and_delta(gpu_device, case, beta):
    """dW = beta dW + Delta^T diag(c_tok) X for bf16 inputs with no stash and no scaled copy: the kernel walks
    the tokens sequence by sequence and re-expresses its accumulators in units of each sequence's
    coefficient.  Coefficients of both signs spanning nine orders of magnitude, exact zeros (their sequences
    are skipped), empty sequences, ragged tails, every launch shape of the sum over all tokens; beta = 0 over
    a NaN-filled dW.  No operand is rounded, so the result is held to the fp32-input tolerance scaled to the
    terms."""
    d_in, d_out, lengths = WEIGHTED_CASES[case]
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=70 + case, sigma_delta=1e-2, rho=0.3)
    layer, _ = to_device(prob, gpu_device)
    rng = np.random.default_rng(90 + case)
    m = prob.n_seq
    c = (rng.standard_normal(m) * 10.0 ** rng.uniform(-6, 3, m)).astype(np.float32)
    c[rng.random(m) < 0.2] = 0.0
    if m > 4:
        c[2] = 0.0
    cd = torch.from_numpy(c).to(gpu_device)
    dW0 = rng.standard_normal((d_out, d_in)).astype(np.float32)
    dW = torch.from_numpy(dW0).to(gpu_device) if beta != 0.0 else torch.full((d_out, d_in), float("nan"),
                                                                           device=gpu_device)
    isopo.weighted_grad(layer, cd, None, beta, dW)
    torch.cuda.synchronize()
    Xo, Do = wl.to_oracle(prob.X), wl.to_oracle(prob.Delta)
    c64 = c.astype(np.float64)
    ref = orc.weighted_grad_tokens(Xo, Do, prob.seq_offsets, c64) + beta * dW0.astype(np.float64)
    mag = orc.weighted_grad_tokens(np.abs(orc.widen(Xo)), np.abs(orc.widen(Do)), prob.seq_offsets, np.abs(c64)) + np.abs(beta * dW0)
    got = dW.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got))
    # fp32 accumulation of exact bf16 products: a few 1e-6 of the terms (atomics of the split add a little)
    assert np.all(np.abs(got - ref) <= 1e-4 * (mag + mag.mean())), f"case {case}: worst {np.max(np.abs(got - ref) / (mag + mag.mean())):.2e}"
    assert_dW_close(got, ref, 1e-4, f"weighted from X, Delta case {case} beta={beta}", mag)
    # all coefficients zero: dW = beta dW exactly
    dW2 = torch.from_numpy(dW0).to(gpu_device) if beta != 0.0 else torch.full((d_out, d_in), float("nan"), device=gpu_device)
    isopo.weighted_grad(layer, torch.zeros(m, device=gpu_device), None, beta, dW2)
    torch.cuda.synchronize()
    assert torch.equal(dW2, torch.from_numpy(dW0).to(gpu_device) * beta if beta != 0.0 else torch.zeros_like(dW2))


def test_weighted_contraction_equals_the_unweighted_one_for_unit_coefficients(gpu_device):
    """c = 1 everywhere: every ratio is one, so the weighted kernel must reproduce the unweighted launch up to the
    zero padding of each sequence's last block (same products, same order within a sequence)."""
    prob = wl.custom_layer(768, 512, [300, 17, 0, 250, 64, 1, 90], dtype="bf16", seed=77, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    ones = torch.ones(prob.n_seq, device=gpu_device)
    a = isopo.weighted_grad(layer, ones)
    b = isopo.weighted_grad(layer, None)
    torch.cuda.synchronize()
    assert torch.allclose(a, b, rtol=1e-5, atol=1e-6 * float(b.abs().max()))


@pytest.mark.parametrize("beta", [0.0, 0.75])
def test_unweighted_contraction_whole_tiles_then_split_tail(gpu_device, beta):
    """More 256x256 output tiles than compute units (17 x 16 = 272, ragged last tile row): the 256 tiles of
    the full round are stored whole, the 16 of the partial round are cut into token chunks and accumulated
    with atomics.  beta = 0 over a NaN-filled dW (must not be read, neither by whole nor by split tiles)
    and beta != 0; every element is compared."""
    d_in, d_out = 4096, 4200
    lengths = [700, 1, 0, 900, 447]
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=37, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    plan = isopo.contraction_plan(layer.ref(), False)
    assert plan["tiles"] == 272 and plan["whole_tiles"] == 256 and plan["n_chunks"] > 1
    rng = np.random.default_rng(8)
    dW0 = rng.standard_normal((d_out, d_in)).astype(np.float32)
    dW = torch.from_numpy(dW0).to(gpu_device) if beta != 0.0 else torch.full((d_out, d_in), float("nan"),
                                                                           device=gpu_device)
    isopo.weighted_grad(layer, None, None, beta, dW)
    torch.cuda.synchronize()
    Xo, Do = wl.to_oracle(prob.X), wl.to_oracle(prob.Delta)
    ones = np.ones(prob.n_seq)
    ref = orc.weighted_grad_tokens(Xo, Do, prob.seq_offsets, ones) + beta * dW0.astype(np.float64)
    mag = orc.weighted_grad_tokens(np.abs(orc.widen(Xo)), np.abs(orc.widen(Do)), prob.seq_offsets, ones) + np.abs(beta * dW0)
    assert_dW_close(dW.cpu().numpy(), ref, TOL["bf16"], f"whole tiles + split tail beta={beta}", mag)


@pytest.mark.parametrize("dims", [(256, 384), (512, 256), (200, 136)])
@pytest.mark.parametrize("beta", [0.0, 0.75])
def test_unweighted_contraction_with_token_split(gpu_device, dims, beta):
    """Few output tiles and many tokens: the sum over all tokens is split into
    token chunks whose partial tiles are accumulated atomically.  Both tile
    sizes, a ragged last chunk, beta = 0 over a NaN-filled dW (must not be read)
    and beta != 0."""
    d_in, d_out = dims
    lengths = [3000, 1400, 1, 4200, 333, 4100]      # 13034 tokens on 2 to 6 output tiles: a dozen or more chunks, the last ragged
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=31, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    rng = np.random.default_rng(6)
    dW0 = rng.standard_normal((d_out, d_in)).astype(np.float32)
    dW = torch.from_numpy(dW0).to(gpu_device) if beta != 0.0 else torch.full((d_out, d_in), float("nan"),
                                                                           device=gpu_device)
    isopo.weighted_grad(layer, None, None, beta, dW)
    torch.cuda.synchronize()
    Xo, Do = wl.to_oracle(prob.X), wl.to_oracle(prob.Delta)
    ones = np.ones(prob.n_seq)
    ref = orc.weighted_grad_tokens(Xo, Do, prob.seq_offsets, ones) + beta * dW0.astype(np.float64)
    mag = orc.weighted_grad_tokens(np.abs(orc.widen(Xo)), np.abs(orc.widen(Do)), prob.seq_offsets, ones) + np.abs(beta * dW0)
    assert_dW_close(dW.cpu().numpy(), ref, TOL["bf16"], f"token split {dims} beta={beta}", mag)


def test_hip_graph_replays_match_eager(gpu_device):
    """The whole layer step (both Gram routes' kernels, the solve, the stash
    sum, the token-sample route) captured in a HIP graph: the library allocates
    nothing, synchronises nowhere and records no memset nodes, so every replay
    must reproduce the eager result for the buffers' current contents."""
    prob = wl.custom_layer(256, 384, [100, 37, 0, 250, 64, 300], dtype="bf16", seed=41, sigma_delta=1e-2)
    layer, A = to_device(prob, gpu_device)
    m = prob.n_seq
    _, full, _ = isopo.gram_plan(layer, "materialised")
    ws = isopo.alloc_workspace(full, gpu_device)
    gws = isopo.alloc_workspace(isopo.gram_plan(layer, "ghost")[1], gpu_device)
    K = torch.empty((m, m), dtype=torch.float32, device=gpu_device)
    Kg = torch.empty_like(K)
    c = torch.empty(m, dtype=torch.float32, device=gpu_device)
    cf = torch.empty_like(c)
    f2 = torch.empty_like(c)
    info = torch.zeros(1, dtype=torch.int32, device=gpu_device)
    dW = torch.empty((prob.d_out, prob.d_in), dtype=torch.float32, device=gpu_device)
    dWf = torch.empty_like(dW)
    dWw = torch.empty_like(dW)
    idx = torch.arange(0, 16 * 40, 40, dtype=torch.int32, device=gpu_device)
    fws = isopo.alloc_workspace(isopo.load().isopo_fisher_samples_workspace(layer.ref(), 16), gpu_device)
    scratch = torch.empty_like(layer.X)

    def run():
        isopo.layer_gram(layer, "materialised", K=K, workspace=ws, keep_stash=True)
        isopo.layer_gram(layer, "ghost", K=Kg, workspace=gws)
        isopo.transform(K, A, "interacting", 1e-2, isopo.REG_REL_TRACE, c=c, info=info)
        isopo.weighted_grad(layer, c, ws, 0.0, dW)
        isopo.fisher_samples(layer, idx, A, 1e-2, isopo.REG_REL_TRACE, cf, f2, fws)
        isopo.weighted_grad_prescaled(layer, cf, scratch, 0.0, dWf)
        isopo.weighted_grad(layer, cf, None, 0.0, dWw)          # the weighted contraction from X and Delta

    def snapshot():
        torch.cuda.synchronize()
        return [t.clone() for t in (K, Kg, c, dW, cf, dWf, dWw)]

    run()                                   # warm-up outside the capture (kernel attributes are set once)
    eager = snapshot()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    A0 = A.clone()
    for rep in range(3):
        A.copy_(A0 * (1.0 + rep))           # the graph reads the buffers' current contents
        for t in (K, Kg, c, dW, cf, dWf, dWw):
            t.fill_(float("nan"))
        graph.replay()
        got = snapshot()
        run()                               # eager work between replays, same inputs
        want = snapshot()
        for name, g, w in zip(("K", "K ghost", "c", "dW", "c samples", "dW samples", "dW samples"), got, want):
            if name == "K ghost":           # fp64 atomics: order varies, one fp32 rounding at most
                assert torch.allclose(g, w, rtol=1e-6, atol=0), f"replay {rep}: {name}"
            elif name == "dW samples":      # may use the token split's fp32 atomics
                assert torch.allclose(g, w, rtol=1e-4, atol=1e-6 * float(w.abs().max())), f"replay {rep}: {name}"
            else:
                assert torch.equal(g, w), f"replay {rep}: {name}"
    assert torch.equal(eager[0], K)         # K does not depend on A
    A.copy_(A0)


@pytest.mark.parametrize("dims,budget", [((512, 768), 8), ((512, 768), 64), ((1024, 512), 224), ((768, 512), 16)])
def test_per_sequence_gradients_on_a_compute_unit_budget(gpu_device, dims, budget):
    """isopo_seq_grads_limited: a launch of `budget` workgroups at most, each of
    which walks a list of (sequence, tile) pairs that the host's plan fixes.  Same
    arithmetic per pair, so the stash must equal the unlimited launch bit for bit -
    with tile counts that are and are not a multiple of eight, ragged and empty
    sequences, and twice in a row on the same scratch words."""
    d_in, d_out = dims
    rng = np.random.default_rng(91)
    n_seq = 80
    lengths = [int(x) for x in rng.integers(0, 120, n_seq)]
    lengths[3] = 0
    prob = wl.custom_layer(d_in, d_out, lengths, dtype="bf16", seed=13, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    plan = isopo.contraction_plan(layer.ref(), True)
    assert plan["tile"] == 256 and plan["workgroups"] > budget
    assert 8 * walk_plan(d_in, d_out, lengths, budget)[0].per_xcd == budget
    ref = isopo.seq_grads(layer)
    queue = torch.full((8,), 12345, dtype=torch.int32, device=gpu_device)       # the call zeroes it
    got = torch.full_like(ref, float("nan"))
    for _ in range(2):
        isopo.seq_grads(layer, got, max_workgroups=budget, queue=queue)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16))
        got.fill_(float("nan"))
    G = orc.seq_logprob_grads(wl.to_oracle(prob.X), wl.to_oracle(prob.Delta), prob.seq_offsets)
    assert rel_err(ref.float().cpu().numpy(), G) < 4e-3
    # a small problem ignores the budget and still answers
    small = wl.custom_layer(64, 64, [5, 9], dtype="bf16", seed=14, sigma_delta=1e-2)
    ls, _ = to_device(small, gpu_device)
    assert torch.equal(isopo.seq_grads(ls, max_workgroups=8).view(torch.int16), isopo.seq_grads(ls).view(torch.int16))
    with pytest.raises(isopo.IsopoError):
        isopo.seq_grads(layer, got, max_workgroups=4, queue=queue)


def test_hip_graph_replays_of_the_persistent_launch(gpu_device):
    """isopo_layer_gram on a layer with more (sequence, tile) pairs than compute
    units, so that a workgroup walks several, captured in a HIP graph: every
    replay, with eager work of the same kind between replays, must reproduce K
    and the stash bit for bit for the buffers' current contents, whatever the
    workspace held before."""
    rng = np.random.default_rng(23)
    lengths = [int(x) for x in rng.integers(1, 90, 96)]
    prob = wl.custom_layer(512, 768, lengths, dtype="bf16", seed=15, sigma_delta=1e-2)
    layer, _ = to_device(prob, gpu_device)
    assert isopo.contraction_plan(layer.ref(), True)["workgroups"] > 256
    _, full, _ = isopo.gram_plan(layer, "materialised")
    ws = isopo.alloc_workspace(full, gpu_device)
    ws_eager = isopo.alloc_workspace(full, gpu_device)
    K = torch.empty((96, 96), dtype=torch.float32, device=gpu_device)
    K_eager = torch.empty_like(K)
    n_stash = isopo.stash_nbytes(layer)

    def run(k, w):
        isopo.layer_gram(layer, "materialised", K=k, workspace=w, keep_stash=True)

    run(K, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(K, ws)
    X0 = layer.X.clone()
    for rep in range(3):
        layer.X.copy_(X0 * (1.0 + rep))     # the graph reads the buffers' current contents
        K.fill_(float("nan"))
        ws.fill_(0xFF)                      # whatever the workspace held
        graph.replay()
        torch.cuda.synchronize()
        run(K_eager, ws_eager)
        torch.cuda.synchronize()
        assert torch.equal(K, K_eager), f"replay {rep}"
        assert torch.equal(ws[:n_stash], ws_eager[:n_stash]), f"replay {rep}: stash"
    layer.X.copy_(X0)
