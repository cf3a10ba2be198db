"""The caching step of rows that keep no key although their CSR row has entries: every column
index out of range (the device CSR was never checked on the host), or every kept score
-inf.  Such rows get rho = 0 and, of the keys that the CSR row does not name, R = the full
output; the other rows are not touched."""

import numpy as np
import pytest

import paper_2505_22918_amd as rt
from oracle import attention as oa
from paper_2505_22918_amd import synth

from parity import assert_bf16_close, assert_stat_close, f64, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [576, 2304])  # the single kernel, and the sparse and dense walks
@pytest.mark.parametrize("D", [64, 72])
@pytest.mark.parametrize("how", ["out of range", "-inf scores"])
@pytest.mark.parametrize("stats", [False, True])
@pytest.mark.filterwarnings("ignore:invalid value", "ignore:divide by zero")
def test_rows_without_a_kept_key(gpu, T, D, how, stats):
    print(f"[no kept key] T={T} D={D} {how} stats={stats}", flush=True)
    n = T // 64
    rng = np.random.default_rng(T + D)
    qkv = [synth.f32_to_bf16_bits(rng.standard_normal((1, 2, T, D), dtype=np.float32)) for _ in range(3)]
    rows = np.arange(4 * 64, 5 * 64)
    left = np.zeros(64, dtype=bool)
    col = np.stack([np.arange(n), np.where(np.arange(n) == 7, 5, 7)], 1)  # two blocks a row
    col.sort(axis=1)
    if how == "out of range":
        left[:] = True
        col[4] = [n, n + 5]
    else:  # block 4 keeps blocks 5 and 6, whose keys are -inf in one dim
        col[4] = [5, 6]
        qkv[1][0, 0, 5 * 64:7 * 64, 9] = 0xFF80
        left = f64(qkv[0])[0, 0, rows, 9] > 0
    mask = rt.BlockMask.from_csr(np.arange(n + 1, dtype=np.int32) * 2, np.clip(col, [0, 1], [n - 2, n - 1]).reshape(-1), 64)
    mask.col_idx.copy_(to_dev_int(col.reshape(-1)))
    got = rt.attn_cache(*(to_dev(x) for x in qkv), mask, stats=stats)
    o, rho, r = (to_np(x)[0, 0, rows] for x in got[:3])
    Q, K, V = (f64(x) for x in qkv)
    of, mf, lf = oa.full_attention_rows(Q, K, V, 0, 0, rows)
    assert left.any() and np.all(rho[left] == 0.0)
    if how == "out of range":  # which keys R sums is left open for a CSR that rt_bsr_check refuses
        assert np.isfinite(r[left]).all()
        return
    assert_bf16_close(r[left], of[left], f"{how} R")
    if stats:
        assert_stat_close(to_np(got[3])[0, 0, rows][left], mf[left], f"{how} m", floor=1.0)
        assert_stat_close(to_np(got[4])[0, 0, rows][left], lf[left], f"{how} l")
    # a row of another block, and the other head's same rows where they keep keys
    assert np.isfinite(to_np(got[2])[0, 1, :4 * 64]).all() and (to_np(got[1])[0, 1, :4 * 64] > 0).all()


def to_dev_int(x):
    import torch

    return torch.from_numpy(np.asarray(x, dtype=np.int32)).cuda()
