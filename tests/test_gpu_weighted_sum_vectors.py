"""The stash's weighted sum at the sizes where the number of vectors a thread takes changes, and at the ragged ends of a
workgroup's vectors, against 64-bit sums."""
import pytest
import torch

from paper_2512_23353_amd import isopo
from paper_2512_23353_amd import workloads as wl

from helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d_in,d_out,m", [
    ("bf16", 1024, 2048, 3),        # 512 workgroups of two vectors
    ("bf16", 1024, 1792, 3),        # 448 of them: too few
    ("bf16", 1024, 2304, 3),        # 576: uneven
    ("bf16", 1000, 2104, 9),        # row-major, the last workgroup a few vectors
    ("bf16", 2040, 4104, 5),
    ("f32", 1028, 1044, 17),
    ("f32", 1000, 1052, 8),
    ("bf16", 4096, 4096, 64),       # 2 GiB: four vectors
    ("bf16", 4096, 4096, 63),
    ("bf16", 3000, 5000, 73),       # row-major past 2 GiB, a ragged end
    ("bf16", 1000, 4192, 6),        # row-major, 1024 workgroups of two vectors
    ("bf16", 1000, 4184, 6),        # 1022: too few
    ("f32", 4096, 3076, 43),        # 2 GiB of wide fp32 sequences: four, a ragged end
    ("f32", 4096, 3068, 43),        # narrower: two
])
@pytest.mark.parametrize("beta", [0.0, -0.5])
def test_weighted_sum_of_stash(gpu_device, dtype, d_in, d_out, m, beta):
    layer, _ = to_device(wl.custom_layer(d_in, d_out, [2] * m, dtype=dtype, seed=m, sigma_delta=1e-2, rho=0.3), gpu_device)
    _, stash = isopo.layer_gram(layer, "materialised", keep_stash=isopo.KEEP_FAST)
    layout = isopo.stash_layout(layer)[0]
    gen = torch.Generator().manual_seed(m)
    c = torch.randn(m, generator=gen).to(gpu_device)
    start = torch.randn((d_out, d_in), generator=gen).to(gpu_device)
    got = isopo.weighted_grad(layer, c, stash, layout=layout, beta=beta, dW=start.clone())
    G, M = beta * start.double(), abs(beta) * start.double().abs()
    for i in range(m):
        r = slice(int(layer.off_host[i]), int(layer.off_host[i + 1]))
        g = layer.Delta[r].double().T.contiguous() @ layer.X[r].double()
        s = layer.Delta[r].double().abs().T.contiguous() @ layer.X[r].double().abs()
        G += c[i].double() * g
        # the stash holds g to its own rounding: 2^-8 of it in bf16, two tokens' sums of six partial products in fp32
        M += c[i].double().abs() * (s + (2.0 ** -9 / 2.0 ** -24 * g.abs() if dtype == "bf16" else 16 * s))
    # each term is added with one rounding, a product with another
    assert ((got.double() - G).abs() <= 2 * (m + 3) * 2.0 ** -24 * M).all()
