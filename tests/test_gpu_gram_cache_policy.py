"""The Gram pass on either side of the stash size up to which its loads stay in the last-level cache (256 MiB)."""
import pytest
import torch

from paper_2512_23353_amd import isopo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n_seq", [(torch.bfloat16, 16), (torch.bfloat16, 100), (torch.float32, 40)])
@pytest.mark.parametrize("over", [0, 8])
def test_gram_at_the_policy_line(gpu_device, dtype, n_seq, over):
    n_elem = (256 << 20) // (n_seq * dtype.itemsize) // 8 * 8 + over
    gen = torch.Generator(device=gpu_device).manual_seed(n_seq)
    S = torch.randn((n_seq, n_elem), generator=gen, device=gpu_device).to(dtype)
    K = isopo.stash_gram(S).double()
    ref, mag = torch.zeros_like(K), torch.zeros_like(K)
    for part in S.split(1 << 20, dim=1):
        p = part.double()
        ref += p @ p.t().contiguous()
        mag += p.abs() @ p.abs().t().contiguous()
    # A workgroup's wave sums its elements in fp32, in chains of 64 in fp32 and of n_elem / 1024 at most in bf16 (exact products);
    # the slots meet in 64 bits.  Roundings of either sign grow like the root of their number; four times that is the bound.
    chain = 64 if dtype == torch.float32 else n_elem / 1024
    assert ((K - ref).abs() <= 4.0 * chain ** 0.5 * 2.0 ** -23 * mag).all()


@pytest.mark.parametrize("dtype,n_seq", [(torch.bfloat16, m) for m in (16, 32, 64, 96, 128, 160, 192, 224, 256)]
                         + [(torch.float32, 16 * b) for b in range(1, 9)])
@pytest.mark.parametrize("over", [0, 8, 136])
def test_gram_of_whole_numbers_at_the_policy_line(gpu_device, dtype, n_seq, over):
    """Every number of row blocks with either policy; entries of -1, 0 and 1 (the last eight of a row none of them 0), so that all
    sums stay below 2^24 and are exact: an element lost, read twice or taken from another row changes K."""
    n_elem = (256 << 20) // (n_seq * dtype.itemsize) // 8 * 8 + over
    gen = torch.Generator(device=gpu_device).manual_seed(n_seq + over)
    S = torch.randint(-1, 2, (n_seq, n_elem), generator=gen, device=gpu_device, dtype=torch.int8)
    S[:, -8:] = 2 * (S[:, -8:] > 0).to(torch.int8) - 1
    ref = torch.zeros((n_seq, n_seq), device=gpu_device, dtype=torch.float64)
    for part in S.split(1 << 20, dim=1):
        p = part.double()
        ref += p @ p.t().contiguous()
    assert float(ref.abs().max()) < 2 ** 24
    assert torch.equal(isopo.stash_gram(S.to(dtype)).double(), ref)
