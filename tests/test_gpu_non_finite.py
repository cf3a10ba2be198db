"""A query row's NaN or infinity stays in that row, and an infinite key reaches only the rows
that it makes infinite.  Rows r and r ^ 32 of a 64-row block share matrix operands in the
two-tile walk (the last 8 dims of a 72-wide head), where a zero times a non-finite value
would carry it over."""

import numpy as np
import pytest

import paper_2505_22918_amd as rt
from oracle import attention as oa
from oracle import block_index as ob
from paper_2505_22918_amd import synth

from parity import assert_bf16_close, assert_stat_close, f64, to_dev, to_np

pytestmark = pytest.mark.gpu

B, H, T, HEAD = 1, 17, 2080, 1  # 1105 waves of 32 rows, 33 blocks: the kernels of long walks
QROW, KROW = 70, 200  # of head HEAD; the key's block (3) is kept by the query's (1)


def _spoil(q, k, D, what):
    """The bf16 bits of one query or key value replaced."""
    kind, dim, bits = {
        "query nan": (q, 3, 0x7FC0), "query tail nan": (q, D - 6, 0x7FC0), "query tail inf": (q, D - 1, 0x7F80),
        "query tail -inf": (q, D - 8, 0xFF80), "key inf": (k, 5, 0x7F80), "key tail inf": (k, D - 2, 0x7F80),
    }[what]
    kind[0, HEAD, QROW if kind is q else KROW, dim] = bits


@pytest.mark.parametrize("what", ["query nan", "query tail nan", "query tail inf", "query tail -inf", "key inf",
                                  "key tail inf"])
@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("call", ["full", "full stats", "sparse", "sparse stats", "reshape", "cache", "cache stats"])
@pytest.mark.filterwarnings("ignore:invalid value")
def test_other_rows_keep_their_values(gpu, call, D, what):
    import torch

    print(f"[non-finite] {call} D={D} {what}", flush=True)
    rng = np.random.default_rng(D)
    qkv = [synth.f32_to_bf16_bits(rng.standard_normal((B, H, T, D), dtype=np.float32)) for _ in range(3)]
    _spoil(qkv[0], qkv[1], D, what)
    n = -(-T // 64)
    hm = np.eye(n, dtype=np.uint8)
    hm[:, 3] = 1
    hm[np.arange(n), (np.arange(n) * 7 + 2) % n] = 1
    rp, ci = ob.block_index_explicit(hm)
    mask = rt.build_index(T, 64, rt.PAT_EXPLICIT, host_mask=hm)
    q, k, v = (to_dev(x) for x in qkv)
    resid = synth.f32_to_bf16_bits(0.1 * rng.standard_normal((B, H, T, D), dtype=np.float32))
    stats = call.endswith("stats")
    kind = call.split()[0]
    if kind == "full":
        got = rt.attn_full(q, k, v, stats=stats)
    elif kind == "sparse":
        got = rt.attn_sparse(q, k, v, mask, stats=stats)
    elif kind == "reshape":
        got = rt.attn_sparse_reshape(q, k, v, mask, torch.full((B, H, T), 0.5, device="cuda"), to_dev(resid))
    else:
        got = rt.attn_cache(q, k, v, mask, stats=stats)
    got = [to_np(x) for x in (got if isinstance(got, tuple) else (got,))]

    Q, K, V = (f64(x) for x in qkv)
    rows = np.arange(64, 128)  # the query's block
    for h in (HEAD, HEAD + 1):
        of, mf, lf = oa.full_attention_rows(Q, K, V, 0, h, rows)
        os_, ms, ls = oa.sparse_attention_rows(Q, K, V, 0, h, rows, rp, ci, 64)
        if kind == "full":
            ref = [of, mf, lf]
        elif kind == "sparse":
            ref = [os_, ms, ls]
        elif kind == "reshape":
            ref = [oa.reshape(os_, np.full(64, 0.5), f64(resid)[0, h, rows], 0.0)]
        else:
            rho = oa.rho(ms, ls, mf, lf)
            ref = [of, rho, oa.residual(of, os_, rho), mf, lf]
        bad = np.isnan(of).any(axis=1)  # the rows that the definitions leave without a value
        assert (bad.sum() > 0) == (h == HEAD) and not bad.all()
        for i, (x, r) in enumerate(zip(got, ref)):
            x = x[0, h, rows]
            assert_close = assert_bf16_close if x.ndim == 2 else assert_stat_close
            kw = {"floor": 1.0} if i == len(ref) - 2 and x.ndim == 1 else {}
            assert_close(x[~bad], r[~bad], f"{call} {what} output {i}", **kw)
            if x.ndim == 2:  # a row without a value has none in any dim
                assert np.isnan(x[bad]).all(), f"{call} {what} output {i}"
