"""The CPU model of the two-tile kernels (tests/kernel_model_tiles.py): addresses and operand
layouts at both head widths over tails of 1 to 64 rows and the largest head, load/wait
schedules of every walk length that the rings treat differently, the caching step's choice
of blocks against its definition, and planted mistakes that must each be caught."""

import numpy as np
import pytest

import kernel_model_tiles as kt

WIDTHS = pytest.mark.parametrize("D", [64, 72])


@WIDTHS
@pytest.mark.parametrize("T", [1, 31, 32, 33, 64, 65, 96, 97, 127, 1000, 17776, "largest"])
def test_addresses(D, T):
    T = (1 << 30) // (2 * D) - 40 if T == "largest" else T
    n = -(-T // 64)
    assert kt.dense_addresses(D, T) == []
    for qb in {0, n // 2, n - 1}:
        assert kt.rows64_addresses(D, T, 64 * qb, sorted({0, qb, n - 1, -1, n, n + 7})) == []


@WIDTHS
@pytest.mark.parametrize("reshape", [False, True])
def test_rows64_schedule(D, reshape):
    for n in list(range(0, 12, 2)) + [62, 64, 66, 128, 130, 556]:
        assert kt.rows64_schedule(D, n, reshape) == [], n


@WIDTHS
def test_dense_schedule(D):
    for n in list(range(1, 10)) + [63, 64, 65, 278]:
        assert kt.dense_schedule(D, n) == [], n


def test_caching_step_scores_the_dropped_blocks():
    rng = np.random.default_rng(3)
    for n in (1, 2, 5, 64, 65, 130, 200):
        for k in {0, 1, n // 2, n - 1, n}:
            kept = sorted(rng.choice(n, size=k, replace=False).tolist())
            assert kt.scored_blocks(kept, n) == sorted(set(range(n)) - set(kept))
            # entries outside the range, as an unchecked CSR may hold, drop no block
            assert kt.scored_blocks([-3, -1] + kept + [n, n + 9], n) == sorted(set(range(n)) - set(kept))
            assert kt.scored_blocks(kept, n, live=False) == []


def test_planted_mistakes_are_caught():
    assert any("before it has landed" in e for e in kt.rows64_schedule(64, 18, True, wait=3))
    assert any("while it is read" in e for e in kt.rows64_schedule(72, 18, True, drain=False))
    assert any("finds" in e for e in kt.rows64_schedule(64, 18, False, swap_v=True))
    assert any("landed" in e for e in kt.dense_schedule(64, 9, in_flight=5))
    assert any("may still read" in e for e in kt.dense_schedule(72, 9, refill_before_barrier=True))
    assert any("not filled" in e for e in kt.rows64_addresses(72, 1000, 0, [0], lanes=16))
    assert kt.rows64_addresses(72, 1000, 0, [0], smem=4 * 32 * 144)
    assert any("filled" in e for e in kt.dense_addresses(72, 1000, rem=8))


def test_planted_layouts_are_caught(monkeypatch):
    # V swizzled as K, and K's tail one slot off
    monkeypatch.setattr(kt.Geo, "vswz", lambda self, r: r & 7 if self.swz else 0 * r)
    dma = kt.Geo.dma
    monkeypatch.setattr(kt.Geo, "dma", lambda self, v: dma(self, False) if not v else kt.LANE * 16)
    assert any("V operand" in e for e in kt.dense_addresses(64, 1000))
    monkeypatch.undo()
    monkeypatch.setattr(kt.Geo, "k_tail", lambda self, q, zero: np.where(kt.HI == q, kt.L32 * self.rowb + 112, zero))
    assert any("K tail" in e for e in kt.rows64_addresses(72, 1000, 0, [0]))
