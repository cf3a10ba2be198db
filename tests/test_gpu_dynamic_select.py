"""The selection of the dynamic mask at the sizes where its kernels change: every count of
64-block tiles a row is selected with in registers (1 to 8), the radix passes above 512
blocks, and the fewest rows a workgroup takes.  Inputs are
small integers, so that every score is exact and many are equal."""

import numpy as np
import pytest

import paper_2505_22918_amd as rt
from oracle import dynamic_mask as dm
from paper_2505_22918_amd import synth

from parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 256, 257, 320, 321, 448, 512, 513, 1300])
def test_selection_at_tile_counts(gpu, D, n):
    B, H, block = 1, 2, 32
    T = n * block
    rng = np.random.default_rng(n + D)
    q, k = (synth.f32_to_bf16_bits(rng.integers(-1, 2, (B, H, T, D)).astype(np.float32)) for _ in range(2))
    k.reshape(B, H, n, block, D)[:, :, ::3] = k.reshape(B, H, n, block, D)[:, :, :1]  # equal blocks: ties
    for keep in sorted({1, 2, min(9, n), max(1, n // 2), max(1, n - 1), n}):
        print(f"[select] D={D} n={n} keep={keep}", flush=True)
        mask = rt.dynamic_index(to_dev(q), to_dev(k), block, keep)
        rp, ci = dm.dynamic_mask(synth.bf16_bits_to_f32(q), synth.bf16_bits_to_f32(k), block, keep)
        assert np.array_equal(mask.row_ptr.cpu().numpy(), rp)
        assert np.array_equal(mask.col_idx.cpu().numpy(), ci)


@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("block", [32, 64])
def test_near_tie_is_ranked_as_the_oracle_does(gpu, D, block):
    """Two keys whose scores are equal with product and sum rounded separately, and one last bit apart
    by fused multiply-adds."""
    from test_oracle_dynamic import near_tie

    print(f"[select] near tie D={D} block={block}", flush=True)
    q, k = near_tie(D, block)
    mask = rt.dynamic_index(*(to_dev(synth.f32_to_bf16_bits(x)[None, None]) for x in (q, k)), block, 2)
    rp, ci = dm.dynamic_mask(q[None, None], k[None, None], block, 2)
    assert list(ci[:2]) == [0, 2]
    assert np.array_equal(mask.col_idx.cpu().numpy(), ci)
