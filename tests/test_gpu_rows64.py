"""Sparse attention and the fused reshape over 64-token blocks, where the walk can go
wrong: rows of 1 to 3 kept blocks (its first and last steps meet), 31 to 34 and 64 to 66
(the offset table is refilled every 64 chunks; the 65th entry is read from memory), a last
block of 1, 32, 33 or 63 tokens, and a row that keeps only that block."""

import numpy as np
import pytest

import paper_2505_22918_amd as rt
from oracle import attention as oa
from oracle import block_index as ob
from paper_2505_22918_amd import synth

from parity import assert_bf16_close, assert_stat_close, f64, sample_rows, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("n,tail", [(1, 1), (2, 33), (3, 32), (5, 63), (70, 1), (70, 64)])
@pytest.mark.parametrize("mode", ["sparse", "sparse stats", "reshape", "reshape stats", "no ratio"])
def test_rows64(gpu, D, n, tail, mode):
    H, T = 2, 64 * (n - 1) + tail
    print(f"[rows64] D={D} T={T} {mode}", flush=True)
    rng = np.random.default_rng(1000 * n + tail)
    hm = np.zeros((H, n, n), dtype=np.uint8)
    for h in range(H):
        for r in range(n):
            keep = [1, 2, 3, 31, 32, 33, 34, 64, 65, 66, n][r % 11]
            hm[h, r, rng.choice(n, size=min(keep, n), replace=False)] = 1
        hm[h, 0] = 0
        hm[h, 0, n - 1] = 1
    mask = rt.build_index(T, 64, rt.PAT_EXPLICIT, host_mask=hm)
    qkv = [synth.f32_to_bf16_bits(rng.standard_normal((1, H, T, D), dtype=np.float32)) for _ in range(3)]
    q, k, v = (to_dev(x) for x in qkv)
    stats = mode.endswith("stats")
    rho = rng.uniform(0.01, 1.0, (1, H, T)).astype(np.float32)
    resid = synth.f32_to_bf16_bits(rng.standard_normal((1, H, T, D), dtype=np.float32))
    if mode.startswith("sparse"):
        got = rt.attn_sparse(q, k, v, mask, stats=stats)
    else:
        import torch

        got = rt.attn_sparse_reshape(q, k, v, mask, None if mode == "no ratio" else torch.from_numpy(rho).cuda(),
                                     to_dev(resid), rho_delta=0.02, stats=stats)
    Q, K, V = (f64(x) for x in qkv)
    for h in range(H):
        rows = sample_rows(rng, T, 64, 200)
        rp, ci = ob.block_index_explicit(hm[h])
        o, m, l = oa.sparse_attention_rows(Q, K, V, 0, h, rows, rp, ci, 64)
        if mode.startswith("reshape"):
            o = oa.reshape(o, rho[0, h, rows].astype(np.float64), f64(resid)[0, h, rows], float(np.float32(0.02)))
        elif mode == "no ratio":
            o = oa.add_residual(o, f64(resid)[0, h, rows])
        out = [to_np(x)[0, h, rows] for x in (got if stats else (got,))]
        assert_bf16_close(out[0], o, f"{mode} O")
        if stats:
            assert_stat_close(out[1], m, f"{mode} m", floor=1.0)
            assert_stat_close(out[2], l, f"{mode} l")
