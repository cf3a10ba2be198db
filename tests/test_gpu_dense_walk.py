"""Dense attention and the caching step over shared K / V rings, where they can go
wrong: last blocks of 1 to 64 tokens, workgroups whose last waves hold no row, both
sides of the rules that choose a kernel, kept sets of one block, many and nearly all
(rows of more than 64 kept blocks included), and non-finite keys and values.
"""

import numpy as np
import pytest

import paper_2505_22918_amd as rt
from oracle import attention as oa
from oracle import block_index as ob
from paper_2505_22918_amd import synth

from parity import assert_bf16_close, assert_stat_close, f64, sample_rows, to_dev, to_np

pytestmark = pytest.mark.gpu

# (B, H, T, D): 1024 waves of 32 rows and one more; 1, 31, 32, 33 and 64 tokens in the last
# block; 1 to 4 waves of the last workgroup with rows; the shortest and a longer walk
SHAPES = [(1, 2, 65, 64), (1, 32, 1024, 64), (1, 33, 1024, 72), (1, 33, 1024, 64), (2, 9, 2049, 64), (1, 17, 2079, 72),
          (1, 16, 2080, 64), (1, 16, 2145, 72), (1, 15, 2304, 64), (1, 5, 4225, 72), (1, 3, 4800, 64)]


def _inputs(B, H, T, D, scale=1.0):
    rng = np.random.default_rng(B * 1000 + H * 100 + T + D)
    return [synth.f32_to_bf16_bits(s * rng.standard_normal((B, H, T, D), dtype=np.float32)) for s in (scale, 1.0, 1.0)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("stats", [False, True])
def test_dense_walk(gpu, shape, stats):
    B, H, T, D = shape
    print(f"[dense] {shape} stats={stats}", flush=True)
    qkv = _inputs(B, H, T, D, 2.0)
    got = rt.attn_full(*(to_dev(x) for x in qkv), stats=stats)
    Q, K, V = (f64(x) for x in qkv)
    rng = np.random.default_rng(1)
    for b, h in ((0, 0), (B - 1, H - 1)):
        rows = sample_rows(rng, T, 64, 96)
        ref = oa.full_attention_rows(Q, K, V, b, h, rows)
        out = [to_np(x)[b, h, rows] for x in (got if stats else (got,))]
        assert_bf16_close(out[0], ref[0], f"{shape} O")
        if stats:
            assert_stat_close(out[1], ref[1], f"{shape} m", floor=1.0)
            assert_stat_close(out[2], ref[2], f"{shape} l")


def _mask(n, keep, rng):
    m = np.zeros((n, n), dtype=np.uint8)
    for r in range(n):
        m[r, rng.choice(n, size=keep, replace=False)] = 1
    return m


@pytest.mark.parametrize("shape", SHAPES[4:] + [(1, 1, 12800, 72), (1, 1, 20000, 64)], ids=str)
@pytest.mark.parametrize("share", ["one", "some", "most"])
@pytest.mark.parametrize("ratio,stats", [(True, True), (True, False), (False, False)])
def test_caching_step(gpu, shape, share, ratio, stats):
    B, H, T, D = shape
    n = -(-T // 64)
    # the rule's limits are 1/8 (D = 64) and 1/3 (D = 72) of the blocks
    keep = {"one": 1, "some": max(1, n // (8 if D == 64 else 3)), "most": n - 1}[share]
    print(f"[cache] {shape} keep={keep} ratio={ratio} stats={stats}", flush=True)
    rng = np.random.default_rng(T + keep)
    hm = _mask(n, keep, rng)
    rp, ci = ob.block_index_explicit(hm)
    mask = rt.build_index(T, 64, rt.PAT_EXPLICIT, host_mask=hm)
    qkv = _inputs(B, H, T, D, 2.0)
    got = rt.attn_cache(*(to_dev(x) for x in qkv), mask, stats=stats, ratio=ratio)
    Q, K, V = (f64(x) for x in qkv)
    for b, h in ((0, 0), (B - 1, H - 1)):
        rows = sample_rows(rng, T, 64, 64)
        of, mf, lf = oa.full_attention_rows(Q, K, V, b, h, rows)
        os_, ms, ls = oa.sparse_attention_rows(Q, K, V, b, h, rows, rp, ci, 64)
        rho = oa.rho(ms, ls, mf, lf)
        r = oa.residual(of, os_, rho) if ratio else oa.residual_no_ratio(of, os_)
        at = lambda x: to_np(x)[b, h, rows]
        assert_bf16_close(at(got[0]), of, f"{shape} O_full")
        assert_bf16_close(at(got[2]), r, f"{shape} R")
        if ratio:
            assert_stat_close(at(got[1]), rho, f"{shape} rho")
        if stats:
            assert_stat_close(at(got[3]), mf, f"{shape} m", floor=1.0)
            assert_stat_close(at(got[4]), lf, f"{shape} l")


@pytest.mark.parametrize("D", [64, 72])
def test_caching_step_keeps_non_finite_values_apart(gpu, D):
    """R sums over the dropped keys only: an infinite V row of a kept block reaches O_full and not R,
    a NaN key of a dropped block reaches R, and rho and R of rows that never meet either
    stay as they are without them."""
    import torch

    T, n = 2304, 36
    hm = np.eye(n, dtype=np.uint8)
    mask = rt.build_index(T, 64, rt.PAT_EXPLICIT, host_mask=hm)
    q, k, v = (to_dev(x) for x in _inputs(1, 4, T, D))
    v2 = v.clone()
    v2[0, 0, 70, 3] = float("inf")  # block 1, head 0
    o, rho, r = rt.attn_cache(q, k, v2, mask, stats=False)
    o0, rho0, r0 = rt.attn_cache(q, k, v, mask, stats=False)
    assert torch.isinf(o[0, 0, :, 3]).all() and torch.equal(rho, rho0)
    assert torch.isfinite(r[0, 0, 64:128]).all() and torch.equal(r[0, 0, 64:128], r0[0, 0, 64:128])
    assert torch.isinf(r[0, 0, :64, 3]).all() and torch.equal(r[0, 1:], r0[0, 1:])
    k2 = k.clone()
    k2[0, 1, 200] = float("nan")  # block 3, head 1
    o, rho, r = rt.attn_cache(q, k2, v, mask, stats=False)
    assert torch.isnan(o[0, 1]).all() and torch.isnan(r[0, 1]).all()
    assert torch.equal(r[0, 0], r0[0, 0]) and torch.equal(rho[0, 2:], rho0[0, 2:])
