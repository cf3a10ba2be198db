"""Dense attention at the lines where its kernel changes: heads of up to 896 tokens in waves of
32 rows or of 64 with a ring each (an odd count of 32-row tiles, 96 / 160 / 224 / 448
tokens, 1024 to 4608 waves), more than 896 tokens, or many heads of 4 blocks, in workgroups
of four waves of which one to four hold rows, or in single waves where those workgroups
need another round, 64-wide heads without statistics at 1024 and 1025 waves of 64 rows."""

import numpy as np
import pytest

import paper_2505_22918_amd as rt
from oracle import attention as oa
from paper_2505_22918_amd import synth

from parity import assert_bf16_close, assert_stat_close, f64, sample_rows, to_dev, to_np

pytestmark = pytest.mark.gpu

# heads, tokens
SHAPES = [(1100, 31), (1100, 32), (600, 33), (600, 64), (400, 65), (400, 96), (400, 97), (300, 128), (300, 129), (300, 160),
          (300, 161), (250, 192), (250, 193), (200, 224), (662, 224), (160, 250), (1024, 250), (1025, 250), (160, 288), (142, 288), (80, 480),
          (32, 1024), (48, 1024), (57, 850), (55, 896), (72, 896), (72, 897), (110, 320), (410, 320), (70, 960), (70, 961),
          (64, 1024), (65, 1024), (62, 1025), (58, 1120), (55, 1180), (16, 4096), (205, 320), (205, 300),
          (64, 1088), (60, 1088), (115, 1088), (125, 1088), (46, 1400)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("stats", [False, True])
def test_dense_lines(gpu, shape, D, stats):
    H, T = shape
    print(f"[dense lines] H={H} T={T} D={D} stats={stats}", flush=True)
    rng = np.random.default_rng(H + T + D)
    qkv = [synth.f32_to_bf16_bits(s * rng.standard_normal((1, H, T, D), dtype=np.float32)) for s in (2.0, 1.0, 1.0)]
    dev = [to_dev(x) for x in qkv]
    got = rt.attn_full(*dev, stats=stats)
    for h in (0, H // 2, H - 1):
        Q, K, V = (f64(x[:, h:h + 1]) for x in qkv)
        rows = sample_rows(rng, T, 64, 64)
        ref = oa.full_attention_rows(Q, K, V, 0, 0, rows)
        out = [to_np(x[:, h])[0, rows] for x in (got if stats else (got,))]
        assert_bf16_close(out[0], ref[0], f"{shape} O")
        if stats:
            assert_stat_close(out[1], ref[1], f"{shape} m", floor=1.0)
            assert_stat_close(out[2], ref[2], f"{shape} l")
    # the tiling does not follow the block argument
    import torch

    again = rt.attn_full(*dev, block=32, stats=stats)
    for x, y in zip(got if stats else (got,), again if stats else (again,)):
        assert torch.equal(x, y)
