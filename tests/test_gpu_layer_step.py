"""The layer step as one call, whose coefficients up to 128 sequences come from the launch that finishes K, against the three calls:
the same bits on either side of the sizes where the launches change, for either Gram path (token products: K to one rounding, and the
coefficients of that K), with a workspace of fewer rows, when replayed from a graph, and with two steps in flight."""
import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo
from paper_2512_23353_amd import workloads as wl

from helpers import to_device

pytestmark = pytest.mark.gpu


def _three_calls(layer, A, variant, lam, path):
    chosen = isopo.gram_plan(layer, path)[0]
    keep = isopo.KEEP_FAST if chosen == "materialised" else 0
    K, ws = isopo.layer_gram(layer, path, keep_stash=keep)
    c, info = isopo.transform(K, A, variant, lam, isopo.REG_REL_TRACE)
    dW = isopo.weighted_grad(layer, c, ws, layout=isopo.stash_layout(layer)[0]) if keep else isopo.weighted_grad(layer, c)
    return dict(K=K, c=c, info=info, dW=dW, path=chosen)


@pytest.mark.parametrize("dtype,m", [("f32", 1), ("f32", 16), ("f32", 17), ("f32", 33), ("f32", 80), ("f32", 128), ("bf16", 2), ("bf16", 16),
                                     ("bf16", 17), ("bf16", 64), ("bf16", 65), ("bf16", 127), ("bf16", 129)])
@pytest.mark.parametrize("variant", ["interacting", "fisher"])
def test_one_call_is_three(gpu_device, dtype, m, variant):
    lens = [(7 * i) % 40 + 1 for i in range(m)]
    layer, A = to_device(wl.custom_layer(264, 328, lens, dtype=dtype, seed=m, sigma_delta=1e-2, rho=0.3), gpu_device)
    want = _three_calls(layer, A, variant, 0.1, "materialised")
    for _ in range(3):                       # whatever the allocator hands out
        got = isopo.layer_step(layer, A, variant, 0.1, isopo.REG_REL_TRACE, "materialised")
        assert got["path"] == "materialised" and got["stash_layout"] == isopo.stash_layout(layer)[0]
        for key in ("K", "c", "info", "dW"):
            assert torch.equal(got[key], want[key]), key


@pytest.mark.parametrize("dtype,d_out,lens", [("bf16", 4096, [33, 0, 128, 1]), ("bf16", 520, [5] * 16), ("bf16", 1032, [3, 40] * 32),
                                              ("bf16", 1032, [9] * 65), ("bf16", 264, [5, 30] * 64), ("bf16", 264, [4] * 130),
                                              ("f32", 328, [20, 0, 31]), ("f32", 328, [7] * 66)])
@pytest.mark.parametrize("variant", ["interacting", "fisher"])
def test_token_products(gpu_device, dtype, d_out, lens, variant):
    """K twice (its 64-bit sums come in any order, so to one rounding), and from the step's own K the same coefficients."""
    layer, A = to_device(wl.custom_layer(512, d_out, lens, dtype=dtype, seed=len(lens), sigma_delta=1e-2, rho=0.3), gpu_device)
    want = _three_calls(layer, A, variant, 0.1, "ghost")
    for _ in range(2):
        got = isopo.layer_step(layer, A, variant, 0.1, isopo.REG_REL_TRACE, "ghost")
        K, ref = got["K"].double(), want["K"].double()
        scale = ref.diagonal().sqrt()
        assert torch.equal(got["K"], got["K"].t()) and got["stash_layout"] is None
        assert ((K - ref).abs() <= 2.0 ** -23 * ref.abs() + 2.0 ** -40 * scale[:, None] * scale[None, :]).all()
        c, info = isopo.transform(got["K"], A, variant, 0.1, isopo.REG_REL_TRACE)
        assert torch.equal(got["c"], c) and torch.equal(got["info"], info)


@pytest.mark.parametrize("m", [3, 70])
def test_not_positive_definite(gpu_device, m):
    """A sequence without tokens and no regulariser: the pivot is named and c is NaN, as from the call by itself."""
    lens = [8] * m
    lens[m // 2] = 0
    layer, A = to_device(wl.custom_layer(256, 256, lens, dtype="bf16", seed=m, sigma_delta=1e-2), gpu_device)
    got = isopo.layer_step(layer, A, "interacting", 0.0, isopo.REG_ABSOLUTE, "materialised")
    want = isopo.transform(got["K"], A, "interacting", 0.0, isopo.REG_ABSOLUTE)
    assert got["info"].item() == want[1].item() > 0 and torch.isnan(got["c"]).all()


def test_replayed(gpu_device):
    layer, A = to_device(wl.custom_layer(256, 512, [40, 7, 0, 90, 33] * 5, dtype="bf16", seed=5, sigma_delta=1e-2, rho=0.3), gpu_device)
    want = isopo.layer_step(layer, A, "interacting", 0.1, isopo.REG_REL_TRACE, "materialised")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = isopo.layer_step(layer, A, "interacting", 0.1, isopo.REG_REL_TRACE, "materialised")
    for _ in range(4):
        for key in ("K", "c", "dW"):
            got[key].fill_(float("nan"))
        got["info"].fill_(77)
        graph.replay()
        other = isopo.layer_step(layer, A, "fisher", 0.1, isopo.REG_REL_TRACE, "materialised")
        torch.cuda.synchronize()
        assert not torch.equal(other["c"], want["c"])
        for key in ("K", "c", "info", "dW"):
            assert torch.equal(got[key], want[key]), key


@pytest.mark.parametrize("dtype,m,d_out", [("bf16", 5, 776), ("bf16", 90, 1032), ("bf16", 130, 520), ("f32", 7, 520), ("f32", 70, 776)])
@pytest.mark.parametrize("variant", ["interacting", "fisher"])
def test_workspace_of_fewer_rows(gpu_device, dtype, m, d_out, variant):
    """A workspace below the full one, whatever it holds: K in several passes over rows, of which each clears the word that the
    workgroups that finish K count in, and dW from X and Delta (few tokens: no atomics).  The three calls on the same workspace, bit for
    bit."""
    layer, A = to_device(wl.custom_layer(264, d_out, [i % 3 // 2 + (m < 20) for i in range(m)], dtype=dtype, seed=m, sigma_delta=1e-2, rho=0.3),
                         gpu_device)
    _, full, least = isopo.gram_plan(layer, "materialised")
    workspace = isopo.alloc_workspace(least, gpu_device)
    assert least < full
    workspace.fill_(0xff)
    K, _ = isopo.layer_gram(layer, "materialised", workspace=workspace)
    c, info = isopo.transform(K, A, variant, 0.1, isopo.REG_REL_TRACE)
    dW = isopo.weighted_grad(layer, c)
    for _ in range(2):
        workspace.fill_(0xff)
        got = isopo.layer_step(layer, A, variant, 0.1, isopo.REG_REL_TRACE, "materialised", workspace=workspace)
        assert got["path"] == "materialised" and got["stash_layout"] is None
        for key, want in (("K", K), ("c", c), ("info", info), ("dW", dW)):
            assert torch.equal(got[key], want), key


def _step(layer, A, path, info, workspace, stream=None):
    """isopo_layer_step as the header has it: the buffers are the caller's, info may be none or shared."""
    full = isopo.gram_plan(layer, path)[1]
    keep = isopo.KEEP_FAST if path == "materialised" and workspace.numel() >= full else 0
    out = dict(K=torch.empty((layer.n_seq, layer.n_seq), device=layer.device), c=torch.full_like(A, float("nan")),
               dW=torch.empty((layer.d_out, layer.d_in), device=layer.device))
    paths = {"ghost": isopo.GRAM_GHOST, "materialised": isopo.GRAM_MATERIALISED}
    status = isopo.load().isopo_layer_step(
        layer.ref(), paths[path], A.data_ptr(), isopo.VARIANT_INTERACTING, 0.1, isopo.REG_REL_TRACE, 0.0, out["K"].data_ptr(),
        out["c"].data_ptr(), None if info is None else info.data_ptr(), out["dW"].data_ptr(), workspace.data_ptr(), workspace.numel(),
        keep, None, None, 0, (stream or torch.cuda.current_stream()).cuda_stream)
    assert status == 0
    return out


@pytest.mark.parametrize("path", ["materialised", "ghost"])
@pytest.mark.parametrize("m", [5, 90])
def test_steps_in_flight(gpu_device, path, m):
    """Two streams, a step on each, one word for the status of both: what a step counts with is in its own workspace.  And none."""
    cases, want = [], []
    for seed in (1, 2):
        layer, A = to_device(wl.custom_layer(256 * seed, 512, [9 * seed] * m, dtype="bf16", seed=seed, sigma_delta=1e-2, rho=0.3), gpu_device)
        workspace = isopo.alloc_workspace(isopo.gram_plan(layer, path)[1], gpu_device)
        cases.append((layer, A, workspace, torch.cuda.Stream()))
        want.append(_three_calls(layer, A, "interacting", 0.1, path))
    info = torch.full((1,), 77, dtype=torch.int32, device=gpu_device)
    torch.cuda.synchronize()
    for word in (info, info, None):
        got = []
        for layer, A, workspace, stream in cases:
            with torch.cuda.stream(stream):
                got.append(_step(layer, A, path, word, workspace, stream))
        torch.cuda.synchronize()
        assert info.item() == 0
        for g, w, (layer, A, _, _) in zip(got, want, cases):
            if path == "materialised":                         # token products: 64-bit sums in any order
                assert torch.equal(g["K"], w["K"]) and torch.equal(g["dW"], w["dW"])
            assert torch.equal(g["c"], isopo.transform(g["K"], A, "interacting", 0.1, isopo.REG_REL_TRACE)[0])
