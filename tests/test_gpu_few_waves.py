"""64-wide heads over 64-token blocks on both sides of the rule that gives few waves attn_fwd
and others attn_rows64: 512 and 513 waves, 1024 with 14 and 15 kept blocks a row, 1408 and
1409, 2048 with 8 and 9, 2049, 6144 and 6145 (with statistics: rows of 3 and 4 blocks), and
the walk's edges with
enough waves for attn_rows64 (rows of 1 to 3 blocks, of 31 to 34 and 64 to 66, last blocks of
1, 32, 33 and 63 tokens)."""

import numpy as np
import pytest

import paper_2505_22918_amd as rt
from oracle import attention as oa
from oracle import block_index as ob
from paper_2505_22918_amd import synth

from parity import assert_bf16_close, assert_stat_close, f64, sample_rows, to_dev, to_np

pytestmark = pytest.mark.gpu
D = 64


def _check(H, T, hm, mode):
    import torch

    n = hm.shape[0]
    print(f"[few waves] {H * n} waves T={T} kept={hm.sum() / n:.1f} {mode}", flush=True)
    rng = np.random.default_rng(T + H)
    mask = rt.build_index(T, 64, rt.PAT_EXPLICIT, host_mask=hm)
    rp, ci = ob.block_index_explicit(hm)
    qkv = [synth.f32_to_bf16_bits(rng.standard_normal((1, H, T, D), dtype=np.float32)) for _ in range(3)]
    resid = synth.f32_to_bf16_bits(rng.standard_normal((1, H, T, D), dtype=np.float32))
    rho = rng.uniform(0.01, 1.0, (1, H, T)).astype(np.float32)
    q, k, v = (to_dev(x) for x in qkv)
    stats = mode.endswith("stats")
    if mode.startswith("sparse"):
        got = rt.attn_sparse(q, k, v, mask, stats=stats)
    else:
        got = rt.attn_sparse_reshape(q, k, v, mask, None if mode == "no ratio" else torch.from_numpy(rho).cuda(),
                                     to_dev(resid), rho_delta=0.02, stats=stats)
    for h in (0, H - 1):
        Q, K, V = (f64(x[:, h:h + 1]) for x in qkv)
        R = f64(resid[:, h:h + 1])[0, 0]
        rows = sample_rows(rng, T, 64, 100)
        o, m, l = oa.sparse_attention_rows(Q, K, V, 0, 0, rows, rp, ci, 64)
        if mode.startswith("reshape"):
            o = oa.reshape(o, rho[0, h, rows].astype(np.float64), R[rows], float(np.float32(0.02)))
        elif mode == "no ratio":
            o = oa.add_residual(o, R[rows])
        out = [to_np(x[:, h])[0, rows] for x in (got if stats else (got,))]
        assert_bf16_close(out[0], o, f"{mode} O")
        if stats:
            assert_stat_close(out[1], m, f"{mode} m", floor=1.0)
            assert_stat_close(out[2], l, f"{mode} l")


def _mask(n, keep):
    rng = np.random.default_rng(n + keep)
    hm = np.zeros((n, n), dtype=np.uint8)
    for r in range(n):
        hm[r, rng.choice(n, size=keep, replace=False)] = 1
    return hm


@pytest.mark.parametrize("H,n,keep", [(32, 16, 2), (27, 19, 2), (32, 32, 14), (32, 32, 15), (88, 16, 3), (1409, 1, 1),
                                      (128, 11, 3), (64, 32, 8), (64, 32, 9), (683, 3, 3), (192, 32, 3), (192, 32, 4),
                                      (1229, 5, 2)])
@pytest.mark.parametrize("mode", ["sparse", "sparse stats", "reshape", "reshape stats"])
def test_both_sides_of_the_rule(gpu, H, n, keep, mode):
    _check(H, 64 * n - 7, _mask(n, keep), mode)


@pytest.mark.parametrize("H,n,tail", [(600, 1, 1), (300, 2, 33), (200, 3, 32), (120, 5, 63), (16, 70, 1), (16, 70, 64)])
@pytest.mark.parametrize("mode", ["sparse", "reshape", "no ratio"])
def test_walk_edges_with_many_waves(gpu, H, n, tail, mode):
    rng = np.random.default_rng(1000 * n + tail)
    hm = np.zeros((n, n), dtype=np.uint8)
    for r in range(n):
        keep = [1, 2, 3, 31, 32, 33, 34, 64, 65, 66, n][r % 11]
        hm[r, rng.choice(n, size=min(keep, n), replace=False)] = 1
    hm[0] = 0
    hm[0, n - 1] = 1
    _check(H, 64 * (n - 1) + tail, hm, mode)
