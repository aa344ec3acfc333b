"""The layout that the product kernels read (csrc/rsr_layout.h), without a GPU: tables packed here by its rules, with none of the
builder's choices of order, are decoded by rsr_export_block's decoder to the paper's index, a numpy walk that mirrors the kernel's
traversal gives the oracle's product, and damaged tables are refused."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle import dense, steps

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
POSITIONS, LANES, WIDE_ROWS, DUMMIES = 48, 64, 256, 32
UNIT = np.dtype([("stream_off", "<u4"), ("block", "<u4"), ("panel", "<u4"), ("heads_lo", "<u4"), ("heads_hi", "<u2"), ("npos", "u1"), ("wide", "u1"),
                 ("units_in_panel", "<u2"), ("extras", "<u2"), ("first", "<u4"), ("reserved", "<u4")])
assert UNIT.itemsize == 32


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("layout") / "layout_shim.so")
    csrc = os.path.join(ROOT, "paper_2411_06360_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=c++20", "-Wall", "-shared", "-fPIC", "-I", csrc, os.path.join(ROOT, "tests", "layout_shim.cpp"),
                    os.path.join(csrc, "rsr_export.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


class Tables:
    """One tile in the layout of rsr_layout.h: segments longer than `cap` rows take eight lanes, a unit holds up to `per_unit` groups."""

    def __init__(self, shim, A, k, cap, per_unit):
        self.A, self.k = A, k
        self.rows, self.cols = A.shape
        self.parts = 2 if (A < 0).any() else 1
        x = np.zeros(5, np.int32)
        shim.shim_shape(ctypes.c_int64(self.rows), k, self.parts, 1, x.ctypes.data_as(ctypes.c_void_p))
        self.kc, self.both, self.pslots, self.nslots, self.panels = map(int, x)
        self.extra_stride = max(2, (self.rows * 2 // WIDE_ROWS + 2) // 2 * 2)
        self.null = self.rows
        halves = steps.ternary_split(A) if self.parts == 2 else (A,)
        blocks = [steps.column_blocks(B, k) for B in halves]
        self.nblocks = len(blocks[0])
        stream, units, self.blk_unit = [], [], [0]
        self.extras = np.zeros((self.nblocks * self.panels, self.extra_stride), np.uint16)
        for b in range(self.nblocks):
            width = blocks[0][b].shape[1]
            vals = [(B[b].astype(np.int64) @ (1 << np.arange(width)[::-1])) << (k - width) for B in blocks]
            for pi in range(self.panels):
                units += self.panel(b, pi, vals, cap, per_unit, stream)
            self.blk_unit.append(len(units))
        self.stream = np.concatenate(stream) if stream else np.zeros(0, np.uint16)
        self.units = np.array(units, UNIT)
        self.blk_unit = np.array(self.blk_unit, np.uint32)

    def panel(self, b, pi, vals, cap, per_unit, stream):
        window_bits = self.k - self.kc
        segments, extra = [], []  # (slot, rows)
        for slot in range(self.nslots):
            low = slot % self.pslots
            part = slot // self.pslots if self.both else pi >> window_bits
            value = low | (0 if self.both else (pi & ((1 << window_bits) - 1)) << self.kc)
            if low >= 1 << self.kc or value == 0:
                continue
            rows = np.flatnonzero(vals[part] == value)
            if len(rows) == 0:
                continue
            pieces = np.array_split(rows, -(-len(rows) // WIDE_ROWS))
            segments.append((slot, pieces[0]))
            for piece in pieces[1:]:
                segments.append((self.nslots + DUMMIES + len(extra), piece))
                extra.append(slot)
        self.extras[b * self.panels + pi, : len(extra)] = extra
        units = []
        for wide, lanes in ((1, 8), (0, 1)):
            ranked = sorted((s for s in segments if (len(s[1]) > cap) == bool(wide)), key=lambda s: -len(s[1]))
            groups = [ranked[i:i + LANES // lanes] for i in range(0, len(ranked), LANES // lanes)]
            taken, positions, heads = 0, [], 0
            for g in groups:
                m = -(-len(g[0][1]) // lanes)
                if positions and (taken == per_unit or len(positions) + m + 1 > POSITIONS):
                    units.append(self.unit(b, pi, wide, positions, heads, stream))
                    taken, positions, heads = 0, [], 0
                rows = np.full((m, LANES), self.null, np.uint16)
                slots = (self.nslots + np.arange(LANES) % DUMMIES).astype(np.uint16)
                for i, (slot, members) in enumerate(g):
                    slots[i * lanes] = slot
                    for j, r in enumerate(members):
                        rows[j // lanes, i * lanes + j % lanes] = r
                positions += list(rows) + [slots]
                heads |= 1 << (len(positions) - 1)
                taken += 1
            if positions:
                units.append(self.unit(b, pi, wide, positions, heads, stream))
        if not units:
            units.append(self.unit(b, pi, 0, [], 0, stream))
        return [u + (len(units), len(extra), 0, 0) for u in units]

    def unit(self, b, pi, wide, positions, heads, stream):
        off = sum(len(s) for s in stream) * 2 // 128
        if len(positions) % 2:
            positions = positions + [np.full(LANES, self.null, np.uint16)]
        p = np.array(positions, np.uint16).reshape(-1, LANES)
        full = len(p) // 8 * 8
        if len(p):
            stream.append(p[:full].reshape(-1, 8, LANES).transpose(0, 2, 1).ravel())   # granules: a lane's 8 positions are adjacent
            stream.append(p[full:].reshape(-1, 2, LANES).transpose(0, 2, 1).ravel())   # rows of dwords
        return (off, b, b * self.panels + pi, heads & 0xffffffff, heads >> 32, len(p), wide)

    def decode(self, shim, part, block):
        width = self.cols - block * self.k if block == self.nblocks - 1 else self.k
        sigma, L, msg = np.full(self.rows, -1, np.int32), np.full((1 << width) + 1, -1, np.int32), ctypes.create_string_buffer(256)
        p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        i64 = ctypes.c_int64
        rc = shim.shim_decode(i64(self.rows), i64(self.cols), self.k, self.parts, p(self.stream), i64(len(self.stream)), p(self.units),
                              i64(len(self.units)), p(self.blk_unit), p(self.extras), i64(self.extras.size), self.extra_stride, part, i64(block),
                              p(sigma), p(L), msg)
        return rc, sigma, L, msg.value.decode()

    def product(self, v):
        """v . A by the kernel's traversal of the tables."""
        act = np.append(v.astype(np.int64), 0)
        out = np.zeros(self.cols, np.int64)
        u = np.zeros((self.nblocks * self.panels, self.nslots + DUMMIES + self.extra_stride), np.int64)
        for U in self.units:
            n, base = int(U["npos"]), int(U["stream_off"]) * 64
            s, full = self.stream[base:base + n * LANES], n // 8 * 8
            pos = np.concatenate([s[:full * LANES].reshape(-1, LANES, 8).transpose(0, 2, 1).reshape(-1, LANES),
                                  s[full * LANES:].reshape(-1, LANES, 2).transpose(0, 2, 1).reshape(-1, LANES)]) if n else s.reshape(0, LANES)
            heads, acc = int(U["heads_lo"]) | int(U["heads_hi"]) << 32, np.zeros(LANES, np.int64)
            for i in range(n):
                if heads >> i & 1:
                    if U["wide"]:
                        acc = np.repeat(acc.reshape(-1, 8).sum(axis=1), 8)
                    u[U["panel"], pos[i]] = acc
                    acc = np.zeros(LANES, np.int64)
                else:
                    acc += act[pos[i]]
        for panel in range(len(u)):
            block, pi = divmod(panel, self.panels)
            n_extra = int(self.units["extras"][self.units["panel"] == panel][0])
            slots = u[panel, : self.nslots].copy()
            for e in range(n_extra):
                slots[self.extras[panel, e]] += u[panel, self.nslots + DUMMIES + e]
            if self.both:
                sign, window, sums = 1, 0, slots[: self.pslots] - slots[self.pslots:]
            else:
                part, window = pi >> (self.k - self.kc), pi & ((1 << (self.k - self.kc)) - 1)
                sign, sums = (-1 if part else 1), slots
            for j in range(1 << self.kc):
                value = window << self.kc | j
                for c in range(min(self.k, self.cols - block * self.k)):
                    if value >> (self.k - 1 - c) & 1:
                        out[block * self.k + c] += sign * sums[j]
        return out


def matrix(kind, rows, cols, seed):
    g = np.random.default_rng(seed)
    if kind == "equal":  # sets of equal rows, some longer than a segment may be
        A = np.repeat(g.integers(-1, 2, size=(5, cols)), [300, 1, 40, 520, 9], axis=0)
        return A[g.permutation(len(A))].astype(np.int8)
    return (g.integers(0, 2, size=(rows, cols)) if kind == "binary" else g.integers(-1, 2, size=(rows, cols))).astype(np.int8)


CASES = [("binary", 300, 17, 4, 47, 3), ("ternary", 257, 21, 7, 12, 99), ("ternary", 130, 30, 12, 6, 2), ("equal", 0, 9, 5, 24, 4),
         ("binary", 5, 13, 13, 47, 1), ("equal", 0, 6, 3, 47, 1)]


@pytest.mark.parametrize("kind,rows,cols,k,cap,per_unit", CASES)
def test_tables_decode_to_the_papers_index_and_give_the_product(shim, kind, rows, cols, k, cap, per_unit):
    A = matrix(kind, rows, cols, 7 * cols + k)
    t = Tables(shim, A, k, cap, per_unit)
    for part, B in enumerate(steps.ternary_split(A) if t.parts == 2 else (A,)):
        for b, Bi in enumerate(steps.column_blocks(B, k)):
            rc, sigma, L, message = t.decode(shim, part, b)
            assert rc == 0, message
            assert np.array_equal(sigma, steps.binary_row_order(Bi))
            assert np.array_equal(L[:-1], steps.full_segmentation(Bi)) and L[-1] == t.rows
    v = np.random.default_rng(3).integers(-128, 128, size=t.rows).astype(np.int8)
    assert np.array_equal(t.product(v), dense.matvec_i8(A, v))


def test_damaged_tables_are_refused(shim):
    A = matrix("equal", 0, 9, 5)
    fresh = lambda: Tables(shim, A, 5, 24, 4)
    t = fresh()
    assert t.decode(shim, 2, 0)[0] != 0 and t.decode(shim, 0, 2)[0] != 0 and t.decode(shim, 0, -1)[0] != 0
    with_rows = int(np.flatnonzero(t.units["npos"] > 8)[0])
    block = int(t.units[with_rows]["block"])
    at = int(t.units[with_rows]["stream_off"]) * 64

    def damage(change):
        d = fresh()
        change(d)
        rcs = [d.decode(shim, p, block) for p in range(d.parts)]
        assert any(rc != 0 and message for rc, _, _, message in rcs), change

    damage(lambda d: d.units["npos"].__setitem__(with_rows, 50))              # more positions than a unit has
    damage(lambda d: d.units["block"].__setitem__(with_rows, block + 1))      # of another block
    damage(lambda d: d.units["units_in_panel"].__setitem__(with_rows, 9))     # the product would wait for units that do not come
    damage(lambda d: d.stream.__setitem__(at, d.rows + 1))                    # a row that is none
    damage(lambda d: d.stream.__setitem__(at, d.stream[at + 1]))              # a row twice
    damage(lambda d: d.units["heads_lo"].__setitem__(with_rows, 0))           # rows that belong to no segment
    damage(lambda d: d.units["extras"].__setitem__(slice(None), 0))           # pieces without a slot
