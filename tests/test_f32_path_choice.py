"""AUTO on fp32 layers takes the Gram path that was measured faster, where the two were apart (no GPU needed)."""
import numpy as np
import pytest

from paper_2512_23353_amd import isopo


@pytest.mark.parametrize("d_in,d_out,n_seq,n_tokens,faster", [
    (300, 1220, 32, 512, "materialised"),       # 39 us against 70
    (1024, 1024, 16, 2400, "materialised"),     # 60 / 240
    (1536, 1536, 8, 128, "materialised"),       # 49 / 112
    (1536, 1536, 32, 2400, "materialised"),     # 177 / 301
    (2048, 4096, 8, 512, "materialised"),       # 179 / 243
    (2048, 4096, 32, 128, "ghost"),             # 440 / 212
    (2048, 4096, 32, 1200, "ghost"),            # 534 / 253
    (2048, 4096, 32, 4800, "materialised"),     # 777 / 2216
])
def test_auto_path(d_in, d_out, n_seq, n_tokens, faster):
    lens = np.full(n_seq, n_tokens // n_seq)
    lens[0] += n_tokens - lens.sum()
    layer = isopo.Layer(None, None, np.concatenate([[0], np.cumsum(lens)]), d_in=d_in, d_out=d_out, dtype=isopo.F32,
                        n_tokens=n_tokens)
    assert isopo.gram_plan(layer, "auto")[0] == faster
    t_ghost, t_materialised = isopo.gram_cost_model(layer)
    assert (t_ghost < t_materialised) == (faster == "ghost") and min(t_ghost, t_materialised) > 0.0
