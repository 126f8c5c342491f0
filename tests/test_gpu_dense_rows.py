"""Rows of 2^17 products and more, and shorter ones that fill their columns,
which go by cells of 2^13 output columns (the heavy rows' units of work otherwise being whole rows), against the
oracle: rows on both sides of a cell's edge, columns on both sides of the
length from which the table of cells holds them (16 entries, 32 in the matrix
of 128 cells), more than 1024 entries in a row, and the same product with the
path switched off.  The library's statistics say how many rows went by cells."""
import numpy as np
import pytest

import oracle
import paper_2608_09713_amd as sp
from paper_2608_09713_amd.workloads import CSR
from tests.parity import compare_full, compare_rows

pytestmark = pytest.mark.gpu

VDT = {"f64": np.float64, "f32": np.float32, "count": None, "jaccard": None}


def _matrix(seed, m, hubs, share, tail, long_rows, last=0):
    """Hub columns held by a share of all rows and the last rows, a few sparse
    entries per row, columns of 15 to 18, 30 to 36 and 60 to 70 entries, and
    long rows of 1500 entries."""
    rng = np.random.default_rng(seed)
    rows, cols = [], []
    for h in range(hubs):
        r = np.flatnonzero((rng.random(m) < share) | (np.arange(m) >= m - last))
        rows.append(r)
        cols.append(np.full(len(r), h))
    rows.append(np.repeat(np.arange(m), tail))
    cols.append(rng.integers(hubs, hubs + 4 * m, m * tail))
    c = hubs + 4 * m
    for ln in [15, 16, 17, 18, *range(30, 37), *range(60, 71)]:
        r = np.unique(rng.integers(0, m - 1, 2 * ln))
        r = np.append(np.sort(rng.choice(r, ln - 1, replace=False)), m - 1)
        rows.append(r)
        cols.append(np.full(ln, c))
        c += 1
    for r in long_rows:
        rows.append(np.full(1500, r))
        cols.append(hubs + rng.choice(4 * m, 1500, replace=False))
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    key = np.unique(rows.astype(np.int64) * (c + 7) + cols)
    rows, cols = key // (c + 7), key % (c + 7)
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=m), out=rp[1:])
    return CSR(m, c + 7, rp, cols.astype(np.int32), rng.standard_normal(len(cols)))


@pytest.mark.parametrize("semiring", ["f64", "f32", "count", "jaccard"])
@pytest.mark.parametrize("m", [16384, 16385, 25000])
def test_dense_rows(semiring, m, monkeypatch):
    A = _matrix(m, m, 24, 0.6, 3, [m - 1, m - 2, 16000])
    A = A.with_values(None if VDT[semiring] is None else A.values.astype(VDT[semiring]))
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    print(f"[{semiring}] m={m} nnz={A.nnz}", flush=True)
    rows = np.unique(np.concatenate([np.arange(0, m, 997), [16000, 16382, 16383, m - 2, m - 1],
                                     np.arange(16384, min(m, 16390))]))
    ref = oracle.lower(A, semiring, rows=rows)
    C = sp.lower(dA, semiring)
    assert 0 < sp.stats()["cell_rows"] <= sp.stats()["heavy_rows"] and sp.stats()["products"] > 1 << 27
    compare_rows(C, ref, rows, semiring, "lower")
    monkeypatch.setenv("SPSYRK_DENSE_ROWS", "0")
    D = sp.lower(dA, semiring)
    assert sp.stats()["cell_rows"] == 0
    monkeypatch.delenv("SPSYRK_DENSE_ROWS")
    assert C.row_ptr.equal(D.row_ptr) and C.col_idx.equal(D.col_idx)
    if VDT[semiring] is None:
        assert C.values.equal(D.values)
    plan, C1 = sp.lower_plan(dA, semiring)
    compare_rows(C1, ref, rows, semiring, "plan")
    if VDT[semiring] is None:
        got, B = plan.execute(None), A
    else:
        B = A.with_values((A.values * 2 - 1).astype(VDT[semiring]))
        got = plan.execute(sp.DeviceCSR.from_host(B, "cuda:0").values)
    compare_rows(got, oracle.lower(B, semiring, rows=rows), rows, semiring, "execute")
    plan.close()


def test_dense_rows_full():
    """Every row of a small matrix whose upper rows are dense."""
    A = _matrix(3, 9000, 40, 0.7, 2, [8999])
    C = sp.lower(sp.DeviceCSR.from_host(A, "cuda:0"), "f64")
    assert sp.stats()["cell_rows"] > 0
    compare_full(C, oracle.lower(A, "f64"), "f64", "lower")


def _cols_shared(m, n, per_row, some):
    """per_row entries of every row in n columns; with some, every third row's in
    40 times as many."""
    rng = np.random.default_rng(m)
    rows, cols = np.repeat(np.arange(m), per_row), rng.integers(0, n, m * per_row)
    if some:
        cols[rows % 3 == 0] += n * rng.integers(1, 41, (rows % 3 == 0).sum())
    key = np.unique(rows * (41 * n) + cols)
    rows, cols = key // (41 * n), key % (41 * n)
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=m), out=rp[1:])
    return CSR(m, 41 * n, rp, cols.astype(np.int32), rng.standard_normal(len(cols)))


@pytest.mark.parametrize("semiring", ["f64", "f32", "count", "jaccard"])
@pytest.mark.parametrize("m, n, per_row, some", [(1400, 600, 200, False), (8193, 3000, 130, True)])
def test_rows_that_fill_their_cells(semiring, m, n, per_row, some, monkeypatch):
    """Rows of 2^14 to 2^17 products: of one cell, and of two (at least 128
    products per entry), beside rows whose columns are too short.  They are
    more than 2^25 products in all; those of the matrix's upper half are fewer
    and stay whole."""
    A = _cols_shared(m, n, per_row, some)
    A = A.with_values(None if VDT[semiring] is None else A.values.astype(VDT[semiring]))
    rp = A.row_ptr
    count = np.zeros(A.ncols, dtype=np.int64)
    products = np.zeros(m, dtype=np.int64)
    for i in range(m):
        c = A.col_idx[rp[i]:rp[i + 1]]
        products[i] = count[c].sum()
        count[c] += 1
    few = (products >= 1 << 14) & (products >= 64 * -(-m // 8192) * np.diff(rp))
    assert products.max() < 1 << 17 and products[few].sum() >= 1 << 25 and few.sum() < m
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    print(f"[{semiring}] m={m} nnz={A.nnz} rows by cells={few.sum()}", flush=True)
    rows = np.unique(np.append(np.arange(0, m, 7), [m // 2 - 1, m - 2, m - 1]))
    ref = oracle.lower(A, semiring, rows=rows)
    C = sp.lower(dA, semiring)
    assert sp.stats()["cell_rows"] == few.sum() < sp.stats()["heavy_rows"]
    compare_rows(C, ref, rows, semiring, "lower")
    monkeypatch.setenv("SPSYRK_DENSE_ROWS", "0")
    D = sp.lower(dA, semiring)
    assert sp.stats()["cell_rows"] == 0
    monkeypatch.delenv("SPSYRK_DENSE_ROWS")
    assert C.row_ptr.equal(D.row_ptr) and C.col_idx.equal(D.col_idx)
    if VDT[semiring] is None:
        assert C.values.equal(D.values)
    plan, C = sp.lower_plan(dA, semiring)
    compare_rows(C, ref, rows, semiring, "plan")
    compare_rows(plan.execute(dA.values), ref, rows, semiring, "execute")
    assert sp.stats()["cell_rows"] == few.sum()
    plan.close()
    h = m // 2
    assert products[:h][few[:h]].sum() < 1 << 25
    U = CSR(h, A.ncols, rp[:h + 1].copy(), A.col_idx[:rp[h]].copy(),
            None if A.values is None else A.values[:rp[h]].copy())
    C = sp.lower(sp.DeviceCSR.from_host(U, "cuda:0"), semiring)
    assert sp.stats()["cell_rows"] == 0
    rows = rows[rows < h]
    compare_rows(C, oracle.lower(U, semiring, rows=rows), rows, semiring, "upper half")


@pytest.mark.parametrize("semiring", ["f64", "count"])
def test_dense_rows_of_many_cells(semiring):
    """128 cells: eight groups of the symbolic pass, offsets over more than 64
    cells, and 32 positions per block of the table of long columns."""
    m, last = 1 << 20, 300
    A = _matrix(20, m, 40, 0.004, 3, [m - 2, m - 700], last)
    A = A.with_values(None if VDT[semiring] is None else A.values)
    assert A.nnz > (1 << 21) + (1 << 14)  # (16 positions per block would be over 2^17 blocks of 128 cells)
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    print(f"[{semiring}] m={m} nnz={A.nnz}", flush=True)
    rows = np.unique(np.concatenate([np.arange(0, m, m // 20), np.arange(m - last, m, 13), [m - 700, m - 2, m - 1]]))
    ref = oracle.lower(A, semiring, rows=rows)
    C = sp.lower(dA, semiring)
    assert sp.stats()["cell_rows"] >= last - 1
    compare_rows(C, ref, rows, semiring, "lower")
    del C
    plan, C = sp.lower_plan(dA, semiring)
    compare_rows(C, ref, rows, semiring, "plan")
    del C
    B = A if VDT[semiring] is None else A.with_values(A.values * 2 - 1)
    got = plan.execute(None if VDT[semiring] is None else sp.DeviceCSR.from_host(B, "cuda:0").values)
    assert sp.stats()["cell_rows"] >= last - 1
    compare_rows(got, oracle.lower(B, semiring, rows=rows), rows, semiring, "execute")
    plan.close()


def test_rows_of_more_lookups_than_products_stay_whole():
    """Four rows of 40,000 entries and four partners each: 160,000 products, but
    128 cells that would each look up every entry."""
    m, wide, ln = 1 << 20, 4, 40000
    rng = np.random.default_rng(5)
    rows = np.concatenate([rng.permutation(m - wide)[:4 * ln], np.repeat(np.arange(m - wide, m), ln)])
    cols = np.concatenate([np.tile(np.arange(ln), 4), np.tile(np.arange(ln), wide)])
    o = np.lexsort((cols, rows))
    rows, cols = rows[o], cols[o]
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=m), out=rp[1:])
    A = CSR(m, ln, rp, cols.astype(np.int32), rng.standard_normal(len(cols)))
    rows = np.concatenate([np.arange(0, m, m // 30), np.arange(m - wide, m)])
    C = sp.lower(sp.DeviceCSR.from_host(A, "cuda:0"), "f64")
    assert sp.stats()["heavy_rows"] == wide and sp.stats()["cell_rows"] == 0
    compare_rows(C, oracle.lower(A, "f64", rows=rows), rows, "f64", "lower")


def test_more_units_than_one_grid_dimension_holds():
    """About 10 M (row, cell) units, past the 2^23 workgroups of 512 threads that
    one grid dimension takes: 2^22 rows (512 cells), the last 24,576 sharing 32
    hub columns.  Counts one-shot, f64 planned and executed."""
    m, last, hubs = 1 << 22, 24576, 32
    rng = np.random.default_rng(8)
    holds = rng.random((last, hubs)) < 0.9
    holds[:, 0] = True
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(holds.sum(1), out=rp[m - last + 1:])
    cols = np.nonzero(holds)[1]
    A = CSR(m, 1000, rp, cols.astype(np.int32), rng.standard_normal(len(cols)))
    products = (np.cumsum(holds, axis=0) - holds)[holds]  # earlier holders of every entry's column
    per_row = np.add.reduceat(products, rp[m - last:m] - rp[m - last])
    assert (per_row >= 1 << 17).sum() * 512 > 1 << 23
    rows = np.concatenate([[0, m - last - 1, m - last, m - last + 5000], np.arange(m - last + 7000, m, 1999), [m - 1]])
    print(f"[units] nnz={A.nnz} dense rows={int((per_row >= 1 << 17).sum())}", flush=True)
    B = A.with_values(None)
    C = sp.lower(sp.DeviceCSR.from_host(B, "cuda:0"), "count")
    assert sp.stats()["cell_rows"] * 512 > 1 << 23
    compare_rows(C, oracle.lower(B, "count", rows=rows), rows, "count", "lower")
    plan, C = sp.lower_plan(sp.DeviceCSR.from_host(A, "cuda:0"), "f64")
    compare_rows(C, oracle.lower(A, "f64", rows=rows), rows, "f64", "plan")
    del C
    B = A.with_values(A.values * 3 + 1)
    compare_rows(plan.execute(sp.DeviceCSR.from_host(B, "cuda:0").values), oracle.lower(B, "f64", rows=rows), rows,
                 "f64", "execute")
    plan.close()
