"""Moves of the running max in the kernels of long calls: dense attention over a shared ring,
the caching step's sparse and dense walks, and the two-tile walk of sparse and fused calls,
at both head widths.

Keys are scaled chunk by chunk, so that scores grow by hundreds to thousands of units during
the walk (steps: many moves; overflow: probabilities pass the fp32 range before a move), or so
that the dropped keys of a caching step score far above the kept ones it starts from, and
the other way round."""

import numpy as np
import pytest

import paper_2505_22918_amd as rt
from oracle import attention as oa
from oracle import block_index as ob
from paper_2505_22918_amd import synth

from parity import assert_bf16_close, assert_stat_close, f64, sample_rows, to_dev, to_np

pytestmark = pytest.mark.gpu

KEPT = (3, 14)  # the key blocks that every row keeps


def _inputs(H, T, D, growth):
    rng = np.random.default_rng(T + D + len(growth))
    q, k, v = (rng.standard_normal((1, H, T, D), dtype=np.float32) for _ in range(3))
    c = np.arange(-(-T // 32))
    kept = np.isin(c // 2, KEPT)
    f = {"steps": 1.0 + 6.0 * c, "overflow": np.where(c % 5 == 4, 80.0, 1.0) * (1.0 + c // 5),
         "dropped above": np.where(kept, 1.0, 40.0), "kept above": np.where(kept, 40.0, 1.0)}[growth]
    k *= np.repeat(f, 32)[:T].astype(np.float32)[None, None, :, None]
    return [synth.f32_to_bf16_bits(x) for x in (q, k, v)]


def _mask(T):
    n = -(-T // 64)
    hm = np.zeros((n, n), dtype=np.uint8)
    hm[:, list(KEPT)] = 1
    return rt.build_index(T, 64, rt.PAT_EXPLICIT, host_mask=hm), ob.block_index_explicit(hm)


def _heads(H, x, T):
    """(head, rows, the oracle's Q, K, V of it) of the first and the last head."""
    rng = np.random.default_rng(T)
    for h in (0, H - 1):
        yield h, sample_rows(rng, T, 64, 100), [f64(y[:, h:h + 1]) for y in x]


@pytest.mark.parametrize("growth", ["steps", "overflow"])
@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("stats", [False, True])
def test_dense(gpu, D, growth, stats):
    H, T = 62, 1030  # 1054 waves of 64 rows, the last workgroup of a head with one of four
    print(f"[rescale long] dense D={D} {growth} stats={stats}", flush=True)
    x = _inputs(H, T, D, growth)
    got = rt.attn_full(*(to_dev(y) for y in x), stats=stats)
    for h, rows, (Q, K, V) in _heads(H, x, T):
        o, m, l = oa.full_attention_rows(Q, K, V, 0, 0, rows)
        at = [to_np(y[:, h])[0, rows] for y in (got if stats else (got,))]
        assert_bf16_close(at[0], o, f"{growth} O")
        if stats:
            assert_stat_close(at[1], m, f"{growth} m", floor=1.0)
            assert_stat_close(at[2], l, f"{growth} l")


@pytest.mark.parametrize("growth", ["steps", "overflow", "dropped above", "kept above"])
@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("stats", [False, True])
def test_caching_step(gpu, D, growth, stats):
    H, T = 3, 2290  # 36 blocks, two of them kept: the sparse and the dense walk
    print(f"[rescale long] cache D={D} {growth} stats={stats}", flush=True)
    x = _inputs(H, T, D, growth)
    mask, (rp, ci) = _mask(T)
    got = rt.attn_cache(*(to_dev(y) for y in x), mask, stats=stats)
    for h, rows, (Q, K, V) in _heads(H, x, T):
        of, mf, lf = oa.full_attention_rows(Q, K, V, 0, 0, rows)
        os_, ms, ls = oa.sparse_attention_rows(Q, K, V, 0, 0, rows, rp, ci, 64)
        rho = oa.rho(ms, ls, mf, lf)
        at = [to_np(y[:, h])[0, rows] for y in got]
        assert_bf16_close(at[0], of, f"{growth} O_full")
        assert_stat_close(at[1], rho, f"{growth} rho", floor=1e-6)
        assert_bf16_close(at[2], oa.residual(of, os_, rho), f"{growth} R")
        if stats:
            assert_stat_close(at[3], mf, f"{growth} m", floor=1.0)
            assert_stat_close(at[4], lf, f"{growth} l")


@pytest.mark.parametrize("growth", ["steps", "overflow"])
@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("stats", [False, True])
def test_sparse_and_fused(gpu, D, growth, stats):
    import torch

    H, T = 35, 990  # 560 waves of 14 kept blocks
    print(f"[rescale long] sparse D={D} {growth} stats={stats}", flush=True)
    x = _inputs(H, T, D, growth)
    n = -(-T // 64)
    hm = np.ones((n, n), dtype=np.uint8)
    hm[np.arange(n), (np.arange(n) + 3) % n] = hm[np.arange(n), (np.arange(n) + 8) % n] = 0
    rp, ci = ob.block_index_explicit(hm)
    mask = rt.build_index(T, 64, rt.PAT_EXPLICIT, host_mask=hm)
    q, k, v = (to_dev(y) for y in x)
    rho = torch.full((1, H, T), 0.4, device="cuda")
    resid = synth.f32_to_bf16_bits(0.05 * np.random.default_rng(1).standard_normal((1, H, T, D), dtype=np.float32))
    sparse = rt.attn_sparse(q, k, v, mask, stats=stats)
    fused = rt.attn_sparse_reshape(q, k, v, mask, rho, to_dev(resid), rho_delta=0.1, stats=stats)
    for h, rows, (Q, K, V) in _heads(H, x, T):
        o, m, l = oa.sparse_attention_rows(Q, K, V, 0, 0, rows, rp, ci, 64)
        y = oa.reshape(o, np.full(len(rows), float(np.float32(0.4))), f64(resid)[0, h, rows], float(np.float32(0.1)))
        for what, got, ref in (("sparse", sparse, o), ("fused", fused, y)):
            at = [to_np(z[:, h])[0, rows] for z in (got if stats else (got,))]
            assert_bf16_close(at[0], ref, f"{growth} {what} O")
            if stats:
                assert_stat_close(at[1], m, f"{growth} {what} m", floor=1.0)
                assert_stat_close(at[2], l, f"{growth} {what} l")
