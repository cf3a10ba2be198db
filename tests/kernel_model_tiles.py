"""CPU model of the two-tile kernels' addressing and load/wait schedule.

Test infrastructure, beside kernel_model.py, for attn_rows64 (csrc/attn.hip) and
attn_dense (csrc/attn_dense.hip) over the walk of csrc/attn_tiles.h.  It restates
the per-lane offsets of their LDS loads, operand reads and epilogues and the
program order of loads, waits, barriers and reads:

* addresses: every loaded 16-byte slot of a ring stage is filled exactly once, with
  the row and head-dim chunk that the operand reads of that place expect; every LDS
  access lies inside the allocation and every global one inside its buffer record or
  wholly past it;
* schedule: every read finds its chunk landed, no load goes into a stage that a
  read may still be on its way from, and, in the shared ring, none into a stage that
  another wave may read between the same two barriers.

It shares nothing with the HIP sources beyond the formulas it restates.
"""

from __future__ import annotations

import numpy as np

LANE = np.arange(64)
L32, HI = LANE & 31, LANE >> 5
G4, L16 = LANE >> 4, LANE & 15
K_OOB = 0x40000000


class Geo:
    def __init__(self, D):
        self.D = D
        self.tail = D == 72
        self.slots = 9 if self.tail else 8  # 16-byte slots of a row
        self.rowb = self.slots * 16
        self.half = 32 * self.rowb
        self.swz = not self.tail

    def kswz(self, r):
        return r & 7 if self.swz else 0 * r

    def vswz(self, r):
        return ((r & 2) << 1) | (r & 1) if self.swz else 0 * r

    def dma(self, v):
        """Byte offset of each lane's 16 bytes in 64 slots of a tensor (v: of V)."""
        if not self.swz:
            return LANE * 16
        r, s = LANE >> 3, LANE & 7
        return r * self.rowb + (s ^ (self.vswz(r) if v else self.kswz(r))) * 16

    # operand reads: LDS offsets within a stage, as the kernel forms them
    def k_read(self, s):
        k_rd = L32 * self.rowb + (HI ^ self.kswz(L32)) * 16
        return k_rd ^ (32 * s) if self.swz else k_rd + 32 * s

    def k_tail(self, q, zero):
        """Offset within the stage in lanes of half q, else the offset of the zeros."""
        return np.where(HI == q, L32 * self.rowb + HI * 16 + 128 - 16 * q, zero)

    def v_read(self, dt, ks):
        r = 4 * HI + (L16 >> 2)
        d = 16 * (L16 & 1) + 8 * (G4 & 1) + 4 * ((L16 >> 1) & 1)
        v_rd = r * self.rowb + ((d >> 3) ^ self.vswz(r)) * 16 + (d & 7) * 2
        return (v_rd ^ (64 * dt) if self.swz else v_rd + 64 * dt) + 16 * ks * self.rowb

    def t_read(self, q, zero):
        t_rd = (16 * (G4 & 1) + 4 * (G4 >> 1) + (L16 >> 2)) * self.rowb + (64 + 4 * (L16 & 1)) * 2
        return np.where(((LANE >> 1) & 1) == q, t_rd, zero)


class Lds:
    """What each 16-byte slot of a stage of `rows` key rows holds: (row, head-dim chunk)."""

    def __init__(self, g, rows):
        self.g = g
        self.row = np.full(rows * g.slots, -1)
        self.chunk = np.full(rows * g.slots, -1)
        self.errors = []

    def load(self, dst, src):
        """16 bytes a lane from source offset src (of the stage's first row) to LDS offset dst."""
        i = dst // 16
        if np.any(dst % 16) or np.any(i < 0) or np.any(i >= len(self.row)):
            self.errors.append("load outside its stage")
            return
        if np.any(self.row[i] != -1) or len(set(i.tolist())) != len(i):
            self.errors.append("slot filled twice")
        self.row[i], self.chunk[i] = src // self.g.rowb, src % self.g.rowb // 16

    def full(self):
        if np.any(self.row < 0):
            self.errors.append("slot not filled")

    def expect(self, at, size, row, dim, what):
        """`size` bytes at LDS offset `at` are head dims dim .. of `row`."""
        if np.any(at < 0) or np.any(at + size > len(self.row) * 16):
            self.errors.append(f"{what}: read outside the stage")
            return
        i, off = at // 16, at % 16
        ok = (off + size <= 16) & (self.row[i] == row) & (8 * self.chunk[i] + off // 2 == dim)
        if not np.all(ok):
            self.errors.append(f"{what}: other data")


def operand_reads(g, k, v, base=0):
    """K and V operand reads of the 32-key chunk whose rows start at `base` of stages k, v."""
    for s in range(4):
        k.expect(base * g.rowb + g.k_read(s), 16, base + L32, 8 * (2 * s + HI), "K operand")
    for dt in range(2):
        for ks in range(2):
            for second in (0, 8):
                r = 16 * ks + second + 4 * HI + (L16 >> 2)
                d = 32 * dt + 16 * (L16 & 1) + 8 * (G4 & 1) + 4 * ((L16 >> 1) & 1)
                v.expect(base * g.rowb + g.v_read(dt, ks) + second * g.rowb, 8, base + r, d, "V operand")
    if g.tail:
        for q in range(2):
            on = HI == q
            at = base * g.rowb + g.k_tail(q, 0)
            k.expect(at[on], 16, base + L32[on], 64, "K tail")
            on = ((LANE >> 1) & 1) == q
            for second in (0, 8):
                at = base * g.rowb + g.t_read(q, 0) + second * g.rowb
                r = 16 * (G4 & 1) + 4 * (G4 >> 1) + (L16 >> 2) + second
                v.expect(at[on], 8, base + r[on], 64 + 4 * (L16[on] & 1), "V tail")


def check_record(errors, offs, record, what):
    """16-byte buffer accesses inside [0, record) or wholly past it (negative offsets are unsigned
    and past every record), below 2^31."""
    offs = np.asarray(offs, np.int64)
    if not np.all((offs + 16 <= 0) | (offs >= record) | ((offs >= 0) & (offs + 16 <= record))):
        errors.append(f"{what}: access straddles the record end")
    if np.any(offs >= 2 ** 31):
        errors.append(f"{what}: offset overflows 32 bits")


# ---- attn_rows64 -------------------------------------------------------------------------


def rows64_loads(g):
    """(LDS offset, source offset adjustment, lanes) of the loads of one chunk."""
    out = [(1024 * m + 16 * LANE, 1024 * m, LANE >= 0) for m in range(4)]
    if g.tail:
        out.append((4096 + 16 * LANE, 4096, LANE < 32))
    return out


def rows64_addresses(D, T, row0, blocks, smem=None, lanes=32):
    """Address checks of one wave: kept key blocks `blocks`, query rows row0 .. (the knobs
    plant a short allocation and another count of lanes in the partial load)."""
    g = Geo(D)
    zero = 4 * g.half
    smem = zero + (8 * g.rowb + 16 if g.tail else 0) if smem is None else smem
    errors = []
    if zero + (8 * g.rowb + 16 if g.tail else 0) > smem:
        errors.append("LDS allocation")
    loads = [(d, a, on if a < 4096 else LANE < lanes) for d, a, on in rows64_loads(g)]
    k, v, r = Lds(g, 32), Lds(g, 32), Lds(g, 32)
    for lds, isv in ((k, False), (v, True), (r, False)):
        for dst, add, on in loads:
            lds.load(dst[on], (g.dma(isv) + add)[on])
        lds.full()
    operand_reads(g, k, v)
    # zeros of the tails: 16 bytes at `zero` and 8 rows on, written by lanes 0 and 1
    # residual rows and outputs, row-wise as K
    for u in range(8):
        at = L32 * g.rowb + ((u ^ g.kswz(L32)) * 16)
        r.expect(at, 16, L32, 8 * u, "residual")
    out = Lds(g, 64)
    for slot in range(64 * g.slots):  # what the epilogue writes: row, chunk at the K layout's place
        row, c = slot // g.slots, slot % g.slots
        out.load(np.array([row * g.rowb + (c ^ int(g.kswz(np.array(row)))) * 16]), np.array([row * g.rowb + c * 16]))
    for m in range(g.slots):
        s = m * 64 + LANE
        row, c = s // g.slots, s % g.slots
        out.expect(row * g.rowb + ((c ^ g.kswz(row)) * 16), 16, row, 8 * c, "output row")
    record, nrow = T * 2 * D, min(T - row0, 64)
    offs = [kb * 64 + 32 * h for kb in blocks for h in range(2)]
    offs = np.array([b * 2 * D if 0 <= b < T else K_OOB for b in offs] + [K_OOB], np.int64)
    for _, add, on in loads:
        for isv in (False, True):
            check_record(errors, offs[:, None] + (g.dma(isv) + add)[on][None, :], record, "K / V load")
        for j in range(2):
            check_record(errors, (g.dma(False) + add)[on] + j * g.half, nrow * 2 * D, "residual load")
    for qt in range(2):
        for s in range(4):
            check_record(errors, (qt * 32 + L32) * 2 * D + (2 * s + HI) * 16, nrow * 2 * D, "Q load")
    return errors + k.errors + v.errors + r.errors + out.errors


class Order:
    """Loads, waits and LDS reads of one wave in program order."""

    def __init__(self):
        self.issued, self.done, self.stage, self.reading, self.errors = [], 0, {}, set(), []

    def issue(self, tag, stage, n):
        if stage in self.reading:
            self.errors.append(f"{tag} goes into {stage} while it is read")
        self.issued += [tag] * n
        self.stage[stage] = (tag, len(self.issued))

    def wait(self, n):
        self.done = max(self.done, len(self.issued) - n)

    def read(self, stage, tag):
        got, end = self.stage.get(stage, (None, 0))
        if got != tag:
            self.errors.append(f"read of {tag} from {stage} finds {got}")
        if end > self.done:
            self.errors.append(f"read of {tag} from {stage} before it has landed")
        self.reading.add(stage)

    def reads_done(self):
        self.reading.clear()


def rows64_schedule(D, n, reshape, wait=2, drain=True, swap_v=False):
    """Program order for n chunks (even); the knobs plant a weaker wait (in chunk loads), a
    missing drain of the reads, and V(i + 2) in the other stage."""
    g, S = Geo(D), Order()
    N = 5 if g.tail else 4
    ktag = lambda c: ("K", c) if c < n else (("R", c - n) if reshape and c - n < 2 else ("past", c))
    vtag = lambda c: ("V", c) if c < n else ("past", c)
    K, V = (lambda c: ("k", c & 1)), (lambda c: ("v", c & 1))
    done = S.reads_done if drain else (lambda: None)
    S.issue("Q", "q", 8 + (2 if g.tail else 0))
    S.issue(ktag(0), K(0), N)
    S.issue(ktag(1), K(1), N)
    S.issue(vtag(0), V(0), N)
    S.wait(wait * N)
    if n:
        S.read(K(0), ("K", 0))
        done()
        S.issue(ktag(2), K(2), N)
        S.issue(vtag(1), V(1), N)
    for i in range(n):
        S.wait(wait * N)
        if i + 1 < n:
            S.read(K(i + 1), ("K", i + 1))
        S.read(V(i), ("V", i))
        if i + 1 < n:
            done()
            S.issue(ktag(i + 3), K(i + 3), N)
            S.issue(vtag(i + 2), V(i + 1 if swap_v else i + 2), N)
    S.wait(0)
    if reshape:
        for qt in range(2):
            S.read(("k", (n + qt) & 1), ("R", qt))
    return S.errors


# ---- attn_dense --------------------------------------------------------------------------

WAVES, STAGES = 4, 3


def dense_loads(g, rem=None):
    """(wave, LDS offset and source adjustment, lanes) of the loads of one 64-row stage."""
    slots = 64 * g.slots
    full = slots // (64 * WAVES)
    rem = (slots - full * 64 * WAVES) // WAVES if rem is None else rem
    out = [(w, (n * WAVES + w) * 1024, LANE >= 0) for n in range(full) for w in range(WAVES)]
    if rem:
        out += [(w, (full * WAVES * 64 + w * rem) * 16, LANE < rem) for w in range(WAVES)]
    return out


def dense_addresses(D, T, rem=None):
    """Address checks of a workgroup over a whole head (rem plants a wrong partial load)."""
    g, errors = Geo(D), []
    k, v = Lds(g, 64), Lds(g, 64)
    loads = dense_loads(g, rem)
    for lds, isv in ((k, False), (v, True)):
        for _, base, on in loads:
            lds.load(base + (16 * LANE)[on], (g.dma(isv) + base)[on])
        lds.full()
    for base in (0, 32):
        operand_reads(g, k, v, base)
    record, blk, n = T * 2 * D, 64 * 2 * D, -(-T // 64)
    for _, base, on in loads:
        x = np.concatenate([np.arange(min(n + 3, 40)), np.arange(max(0, n - 3), n + 3)]).astype(np.int64) * blk
        check_record(errors, x[:, None] + (g.dma(False) + base + g.half)[on][None, :], record, "K load")
        check_record(errors, x[:, None] + (g.dma(True) + base)[on][None, :], record, "V load")
        first = (g.dma(False) + base - g.half)[on]  # block 0's first half, behind 32 rows of zeros
        check_record(errors, first, record, "first K load")
    # zeros: V of blocks not scored (a chunk from `zero` on) and the tails' operands
    zlen = g.half + 256
    for dt in range(2):
        for ks in range(2):
            if np.any(g.v_read(dt, ks) + 8 * g.rowb + 8 > zlen):
                errors.append("zero V operand outside")
    if g.tail and np.any(g.t_read(0, 0) + 8 * g.rowb + 8 > zlen):
        errors.append("zero V tail outside")
    return errors + k.errors + v.errors


def dense_schedule(D, n, in_flight=2, refill_before_barrier=False):
    """Between two barriers a wave may be anywhere: reads and loads of one interval must not share
    a stage, and what an interval reads every wave has waited for before its first barrier.
    The knobs plant a weaker wait (in loads of one stage and tensor) and a refill that does not
    wait for the other waves."""
    N = len([1 for w, _, _ in dense_loads(Geo(D)) if w == 0])  # loads of a wave per stage and tensor
    errors, issued, landed = [], [], 0
    stage = {}  # stage -> (what it holds, its last load's index)
    reads, loads = set(), set()

    def issue(st, tag, n_load):
        nonlocal issued
        loads.add(st)
        if st in reads:
            errors.append(f"{tag} goes into stage {st}, which a wave may still read")
        issued += [tag] * n_load
        stage[st] = (tag, len(issued))

    def barrier():
        reads.clear()
        loads.clear()

    def wait(k):
        nonlocal landed
        landed = max(landed, len(issued) - k)

    ready = 0  # loads that every wave has waited for before the last barrier

    def read(st, tag):
        reads.add(st)
        got, end = stage.get(st, (None, 0))
        if got != tag or st in loads:
            errors.append(f"read of {tag} in stage {st} finds {got}")
        if end > ready:
            errors.append(f"read of {tag} before every wave's part has landed")

    def sync():
        nonlocal ready
        ready = landed
        barrier()

    issue(2, "first", N)
    issue(0, 0, 2 * N)
    issue(1, 1, 2 * N)
    wait(in_flight * N)
    sync()
    read(2, "first")
    sync()
    issue(2, 2, 2 * N)
    st = 0
    for p in range(n):
        read(st, p)
        if refill_before_barrier:
            issue(st, p + 3, 2 * N)
        wait(in_flight * N)
        sync()
        if not refill_before_barrier:
            issue(st, p + 3, 2 * N)
        st = (st + 1) % STAGES
    return errors


def scored_blocks(kept, n, live=True):
    """The blocks that a wave of the caching step scores, as the kernel's generator walks a CSR
    row (ascending entries, some perhaps outside [0, n))."""
    out, k_i, n_kept = [], 0, len(kept)
    entry = lambda i: -1 if i >= n_kept else kept[i]
    k_next = entry(0)
    for c in range(n):
        act = True
        if k_i < n_kept:
            while k_next < c:
                k_i += 1
                if k_i >= n_kept:
                    break
                k_next = entry(k_i)
            if k_i < n_kept and k_next == c:
                act = False
                k_i += 1
                k_next = entry(k_i)
        if act and live:
            out.append(c)
    return out
