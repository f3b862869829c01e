"""Host model of the batch walk (csrc/batch.hpp): the parts of a slice, their
batches, the rowptr windows and the passes over row segments, re-enacted on many
CSR shapes.  Every nonzero of a part is passed once, in a pass of its own row;
every row end is written exactly once, partial rows go through the slice's own
slots, each of them written by one part, and every index stays inside its array."""
import os
import re

import numpy as np
import pytest

from tests.test_partition import slice_bounds, slice_len, snap_len


def index(x):
    """The kernel's row and nonzero counters: unsigned, 32 bits."""
    return x & 0xFFFFFFFF


class Walk:
    def __init__(self, rowptr, N, i0, p0, i1, p1, cap, last=True):
        self.rp, self.N, self.i0, self.p0, self.i1, self.p1 = rowptr, N, i0, p0, i1, p1
        self.cap, self.last = cap, last
        self.head = i0 < i1 and p0 > rowptr[i0]
        self.rlast = i1 if i1 < N else i1 - 1

    def window(self, rb):
        ws, we = [], []
        for lane in range(64):
            r = index(rb + lane)
            if r <= self.rlast:
                assert rb <= r < self.N  # reads rowptr[r], rowptr[r + 1]
                ws.append(max(int(self.rp[r]), self.p0))
                we.append(min(int(self.rp[r + 1]), self.p1))
            else:
                ws.append(0)
                we.append(0)
        return ws, we

    def passes(self, ib, pb, pe, npp):
        """Yields (p, n, row, first, last, cont, open)."""
        rb = ib
        while True:
            ws, we = self.window(rb)
            for b in range(64):
                s, e = max(ws[b], pb), min(we[b], pe)
                p = s
                while p < e:  # p is compared past the row's end, too
                    n = min(npp, e - p)
                    row = rb + b
                    yield (p, n, row, p == s, p + n == e, ws[b] < pb,
                           row == self.i1 or we[b] > pe)
                    p = index(p + npp) if index(p + npp) < e else e
            if not (index(rb + 63) < self.rlast and we[63] < pe):
                return
            rb = index(rb + 64)

    def run(self, npp, y, A, written, slots):
        """One column: A[row] or the slice's head / tail slot gets the sums."""
        dest = lambda r: "t" if r == self.i1 else "h" if r == self.i0 and self.head else r  # noqa: E731

        def put(d, v):
            if isinstance(d, str):
                slots[d] = v
            else:
                assert written[d] == 0
                A[d], written[d] = v, 1

        rb = self.i0
        while rb <= self.rlast:
            ws, we = self.window(rb)
            for b in range(64):
                if index(rb + b) <= self.rlast and rb + b != self.i1 and we[b] <= ws[b]:
                    put(dest(rb + b), 0.0)
            rb = index(rb + 64)
        ib, pb, crow, seen = self.i0, self.p0, -1, []
        while pb < self.p1:
            pe = min(self.p1, pb + self.cap)
            inext, orow = ib, -1  # the row that goes on in the next batch, if any
            if pe < self.p1:
                while inext <= self.rlast:
                    ws, we = self.window(inext)
                    m = [b for b in range(64) if index(inext + b) <= self.rlast and we[b] > pe]
                    if m:
                        inext += m[0]
                        if ws[m[0]] < pe:
                            orow = inext
                        break
                    inext = index(inext + 64)
                assert inext <= self.rlast
            acc = 0.0
            for p, n, row, first, last, cont, opened in self.passes(ib, pb, pe, npp):
                assert pb <= p and p + n <= pe and p + n - pb <= self.cap
                assert self.rp[row] <= p and p + n <= self.rp[row + 1]
                assert cont == (row == crow) and opened == (row in (self.i1, orow))
                if first:
                    assert acc == 0.0
                seen += range(p, p + n)
                acc += float(y[p:p + n].sum())
                if last:
                    d = dest(row)
                    if cont:
                        acc += slots[d] if isinstance(d, str) else A[d]
                    if opened and not isinstance(d, str):
                        A[d] = acc  # the row of A itself holds the sum of its first batches
                    else:
                        put(d, acc)
                    acc = 0.0
            ib, crow, pb = inext, orow, pe
        assert seen == list(range(self.p0, self.p1))
        if self.last and self.i1 < self.N and self.p1 <= self.rp[self.i1]:
            slots["t"] = 0.0


def shapes():
    rng = np.random.default_rng(7)
    out = {"one": [1], "empty": [0] * 200, "none_then_one": [0] * 130 + [1], "long": [0, 5000, 0, 0, 3],
           "ones": [1] * 700, "hub_mid": [2] * 90 + [9000] + [0] * 70 + [1] * 5,
           # a slice that ends at the start of a long row, after rows that cross batches
           "empty_tail": [99] * 10 + [2999], "window_edges": ([3] * 63 + [0]) * 6 + [70] * 130,
           "power": np.minimum((rng.pareto(1.1, 1500) * 3 * (rng.random(1500) < 0.6)).astype(int), 4000)}
    return out.items()


def part(rowptr, N, nnz, S, k, q, parts):
    """make_part: coordinates of part q of slice k and, of the first part, the head row."""
    d0, d1 = k * S, min(k * S + S, N + nnz)
    snap = snap_len(S)

    def cut(d, ref):
        lo = max(0, d - nnz)
        i = max(x for x in range(lo, min(d, N) + 1) if rowptr[x] + x <= d)
        if i >= N:
            return i, nnz
        r0, r1 = int(rowptr[i]), int(rowptr[i + 1])
        return i, (ref - i if r0 + i < ref and r1 - r0 > snap else r0)

    i0, p0 = cut(min(d0 + S * q // parts, d1), d0)
    i1, p1 = cut(min(d0 + S * (q + 1) // parts, d1), d1 if q + 1 == parts else d0)
    head = -1
    if q == 0 and i0 < N and p0 > rowptr[i0] and rowptr[i0 + 1] + i0 + 1 <= d1:
        head = i0
    return i0, p0, i1, p1, head


@pytest.mark.parametrize("parts", [1, 3, 5, 31])
@pytest.mark.parametrize("workers", [1, 3, 40])
@pytest.mark.parametrize("name,lengths", shapes())
def test_parts_of_a_slice(name, lengths, workers, parts):
    lengths = lengths[:700]
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    N, nnz = len(lengths), int(rowptr[-1])
    y = np.random.default_rng(1).integers(1, 9, nnz).astype(float)
    S = slice_len(N + nnz, workers, 64, N=N, nnz=nnz)
    A, written, open_row = np.zeros(N), np.zeros(N, int), None
    for k in range(-(-(N + nnz) // S)):
        at = slice_bounds(rowptr, N, nnz, S, k * S, snap_len(S))
        end = slice_bounds(rowptr, N, nnz, S, min(k * S + S, N + nnz), snap_len(S))
        slots, heads, head_row = {}, [], -1
        for q in range(parts):
            i0, p0, i1, p1, h = part(rowptr, N, nnz, S, k, q, parts)
            assert (i0, p0) == at and (i1, p1) >= at  # parts follow one another
            at, last = (i1, p1), q + 1 == parts
            if q == 0:
                head_row = h
            w = Walk(rowptr, N, i0, p0, i1, p1, 64, last)
            heads += [i0] if w.head else []
            mine = {}
            w.run(8, y, A, written, mine)
            assert last or "t" not in mine
            assert not slots.keys() & mine.keys()
            slots.update(mine)
        assert at == end and heads == ([head_row] if head_row >= 0 else [])
        if head_row >= 0:
            assert open_row is not None and open_row[0] == head_row and written[head_row] == 0
            A[head_row], written[head_row] = open_row[1] + slots["h"], 1
            open_row = None
        if end[0] < N:
            base = open_row[1] if open_row and open_row[0] == end[0] else 0.0
            open_row = (end[0], base + slots["t"])
    assert written.all()
    assert np.array_equal(A, [y[a:b].sum() for a, b in zip(rowptr, rowptr[1:])])


@pytest.mark.parametrize("cap", [64, 512])
@pytest.mark.parametrize("workers", [1, 4, 7, 200])
@pytest.mark.parametrize("name,lengths", shapes())
def test_every_nonzero_and_row_once(name, lengths, workers, cap):
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    N, nnz = len(lengths), int(rowptr[-1])
    y = np.random.default_rng(1).integers(1, 9, nnz).astype(float)
    S = slice_len(N + nnz, workers, 64, N=N, nnz=nnz)
    ns = -(-(N + nnz) // S)
    bounds = [slice_bounds(rowptr, N, nnz, S, min(k * S, N + nnz), snap_len(S)) for k in range(ns + 1)]
    for npp in (1, 8, 16):
        A, written, open_row = np.zeros(N), np.zeros(N, int), None
        for (i0, p0), (i1, p1) in zip(bounds, bounds[1:]):
            w, slots = Walk(rowptr, N, i0, p0, i1, p1, cap), {}
            w.run(npp, y, A, written, slots)
            if w.head:  # the row that earlier slices left open ends here
                assert open_row is not None and open_row[0] == i0 and written[i0] == 0
                A[i0], written[i0] = open_row[1] + slots["h"], 1
                open_row = None
            if i1 < N:
                assert "t" in slots
                base = open_row[1] if open_row and open_row[0] == i1 else 0.0
                open_row = (i1, base + slots["t"])
        assert written.all()
        assert np.array_equal(A, [y[a:b].sum() for a, b in zip(rowptr, rowptr[1:])])


BATCH_TILE, BATCH_L = 64, 512  # kBatchTile, kBatchL


def batch_tile(width):
    q4 = -(-width // 4)
    n = -(-q4 // BATCH_TILE)
    return -(-q4 // n) if n else 1


def tiles_of_launches(L):
    """Columns that the lanes of each tile of each launch store, as run_walk and BatchWalk::rows cut them."""
    for l0 in range(0, L, BATCH_L):
        Lw = min(L - l0, BATCH_L)
        q4, tl = -(-Lw // 4), batch_tile(Lw)
        for q0 in range(0, q4, tl):
            cols = set()
            for q in range(min(tl, q4 - q0)):
                first = 4 * (q0 + q)
                valid = Lw - first
                col = Lw - 4 if valid < 4 <= Lw else first
                cols.update(range(l0 + col, l0 + col + (4 if Lw >= 4 else valid)))
            yield cols


def test_no_column_in_two_tiles():
    # a row's sums are added to A tile by tile: a column in two of them would be added twice
    for L in range(1, 3000):
        seen = [c for cols in tiles_of_launches(L) for c in cols]
        assert sorted(seen) == list(range(L)), L


class At(dict):
    """A long array that is held only where it matters: 0 elsewhere."""
    def __missing__(self, i):
        return 0


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 130])
def test_rows_up_to_the_index_limit(rows):
    N = (1 << 31) - 2 - rows % 3
    rp = At({N: 1})
    A, written = At(), At()
    w = Walk(rp, N, N - rows, 0, N, 1, 512)
    w.run(8, np.ones(1), A, written, {})
    assert sorted(written) == list(range(N - rows, N)) and A[N - 1] == 1.0


@pytest.mark.parametrize("npp", [1, 16])
def test_nonzeros_up_to_the_index_limit(npp):
    nnz = (1 << 31) - 2
    w = Walk([0, nnz], 1, 0, nnz - 700, 1, nnz, 512)
    w.head = False  # the last slice of the row, without its carry
    p = [x for pb, pe in ((nnz - 700, nnz - 188), (nnz - 188, nnz)) for x in w.passes(0, pb, pe, npp)]
    assert sum(x[1] for x in p) == 700 and p[-1][0] + p[-1][1] == nnz


def test_phases_that_exchange_data_are_ordered():
    """Between two phases of a batch in which one lane writes what another reads (the batch
    in LDS, the dots beside it, the rows of A that go on in the next batch) stands an
    ordering of the wave's memory operations."""
    src = os.path.join(os.path.dirname(__file__), "..", "paper_2205_11622_amd", "csrc", "batch.hpp")
    with open(src) as f:
        run = f.read().split("void run(const Part &s)")[1]
    phases = [r"nz\[t \* 64 \+ lane\] = z\[t\];", r"dots<64>\(", r"float y = .*nz\[t\]\.y", r"rows<64>\(", r"pb = pe;"]
    at = [re.search(p, run).start() for p in phases]
    assert at == sorted(at)
    for a, b in zip(at, at[1:]):
        assert "lanes_ordered();" in run[a:b], run[a:b]
