"""Light rows at the edges of their size classes, against the oracle.

A light row's products are sorted in 8, 16, 32 or 64 lanes, in two registers
or, past 128, in LDS; keys are 32 or (plus-times past 2^23 output columns,
Jaccard values staged unpacked) 64 bits; plus-times values come from the
column index or, where it keeps entries, from A by entry.
"""
import numpy as np
import pytest

import oracle
import paper_2608_09713_amd as sp
from paper_2608_09713_amd.workloads import CSR
from tests.parity import compare_full

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 66, 127, 128, 129, 130, 191, 192, 193, 255, 256, 257,
         320, 384, 447, 511, 512]
VDT = {"f64": np.float64, "f32": np.float32, "count": None, "jaccard": None}


def _rows(seed, base_rows, spread, repeats, spare):
    """A whose last rows have SIZES[k] products with the first base_rows (every
    spread-th row): private columns per row, each with a run of base rows, the
    runs disjoint (repeats False) or drawn with repeats.  spare: empty columns
    between the used ones."""
    rng = np.random.default_rng(seed)
    sizes = [p for p in SIZES for _ in range(3)]
    rng.shuffle(sizes)
    m = base_rows * spread + len(sizes)
    rows, cols, col = [], [], 0
    for k, p in enumerate(sizes):
        order = rng.permutation(base_rows)
        done = 0
        while done < p:
            # (long runs for the larger rows: at most 256 entries in a light row)
            ln = int(min(p - done, rng.integers(1, 2 + p // 24 + 6)))
            part = rng.choice(base_rows, ln, replace=False) if repeats else order[done:done + ln]
            rows += list(part * spread) + [base_rows * spread + k]
            cols += [col] * (ln + 1)
            done += ln
            col += 1 + spare
    ncols = max(col, 1) + 5
    rows, cols = np.array(rows, dtype=np.int64), np.array(cols, dtype=np.int64)
    o = np.lexsort((cols, rows))
    rows, cols = rows[o], cols[o]
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=m), out=rp[1:])
    return CSR(m, ncols, rp, cols.astype(np.int32), rng.standard_normal(len(cols))), base_rows * spread


def _as(A, semiring):
    return A.with_values(None if VDT[semiring] is None else A.values.astype(VDT[semiring]))


def _part(A, lo, hi):
    e0, e1 = A.row_ptr[lo], A.row_ptr[hi]
    return CSR(hi - lo, A.ncols, A.row_ptr[lo:hi + 1] - e0, A.col_idx[e0:e1], A.values[e0:e1])


@pytest.mark.parametrize("semiring", ["f64", "f32", "count", "jaccard"])
@pytest.mark.parametrize("repeats", [False, True])
@pytest.mark.parametrize("spread,pack,entries", [(1, "1", False), (1, "0", True), ((1 << 23) // 600 + 1, "0", True)])
def test_size_classes(semiring, repeats, spread, pack, entries, monkeypatch):
    monkeypatch.setenv("SPSYRK_PACK_STAGING", pack)
    monkeypatch.setenv("SPSYRK_LOCAL_SORT", "1" if entries else "0")
    A, split = _rows(11 + repeats, 600, spread, repeats, spare=4 if entries else 0)
    A = _as(A, semiring)
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    print(f"[{semiring}] m={A.nrows} n={A.ncols} nnz={A.nnz} repeats={repeats}", flush=True)
    ref = oracle.lower(A, semiring)
    C = sp.lower(dA, semiring)
    assert sp.stats()["light_rows"] > 0
    compare_full(C, ref, semiring, "lower")
    again = sp.lower(dA, semiring)
    assert again.values.equal(C.values) or sp.stats()["heavy_rows"] > 0  # light rows are reproducible
    plan, C1 = sp.lower_plan(dA, semiring)
    compare_full(C1, ref, semiring, "plan")
    if VDT[semiring] is None:
        compare_full(plan.execute(None), ref, semiring, "execute")
    else:
        B = A.with_values((A.values * 3 - 1).astype(VDT[semiring]))
        got = plan.execute(sp.DeviceCSR.from_host(B, "cuda:0").values)
        compare_full(got, oracle.lower(B, semiring), semiring, "execute")
    plan.close()
    # off the diagonal: the listed rows against all rows (no pruning)
    T = _part(A.with_values(np.zeros(A.nnz) if A.values is None else A.values), split, A.nrows)
    T = T.with_values(None if A.values is None else T.values)
    D = sp.offdiag(sp.DeviceCSR.from_host(T, "cuda:0"), dA, semiring)
    compare_full(D, oracle.offdiag(T, A, semiring), semiring, "offdiag")


@pytest.mark.parametrize("semiring", ["f64", "f32"])
@pytest.mark.parametrize("dense", [False, True])
def test_index_of_entries(semiring, dense, monkeypatch):
    """The index that keeps entries in place of values: fewer products than
    entries, and more (hub columns, also heavy rows), where it is split into
    keys and values after all; one-shot and planned."""
    monkeypatch.setenv("SPSYRK_LOCAL_SORT", "1")
    rng = np.random.default_rng(5)
    m, n, d = 3000, 70000, 12
    D = np.sort(rng.choice(n, (m, d)), axis=1)
    if dense:
        D[:, 0] = rng.integers(0, 4, m)  # four hub columns: every row meets hundreds of others
        D[:40, 1] = 7
        D = np.sort(D, axis=1)
    keep = np.ones(D.shape, dtype=bool)
    keep[:, 1:] = D[:, 1:] != D[:, :-1]
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(keep.sum(1), out=rp[1:])
    A = CSR(m, n, rp, D[keep].astype(np.int32), rng.standard_normal(int(rp[-1])).astype(VDT[semiring]))
    assert A.nnz <= A.ncols
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    C = sp.lower(dA, semiring)
    st = sp.stats()
    assert (st["products"] > A.nnz) == dense and (st["heavy_rows"] > 0) == dense
    compare_full(C, oracle.lower(A, semiring), semiring, "lower")
    plan, _ = sp.lower_plan(dA, semiring)
    for k in range(2):
        B = A.with_values((A.values * (k + 2) + 1).astype(VDT[semiring]))
        got = plan.execute(sp.DeviceCSR.from_host(B, "cuda:0").values)
        compare_full(got, oracle.lower(B, semiring), semiring, f"execute {k}")
    plan.close()


@pytest.mark.parametrize("semiring", ["f64", "jaccard"])
@pytest.mark.parametrize("m", [98303, 98304, 100001])
def test_chunks_dealt_and_counted(semiring, m, monkeypatch):
    """One row per chunk: the most chunks that are dealt out in turn, and the
    fewest that are taken from a counter; lower (32-bit keys) and off the
    diagonal (Jaccard: 64-bit keys, fewer wavefronts)."""
    monkeypatch.setenv("SPSYRK_ROWS_PER_CHUNK", "1")
    rng = np.random.default_rng(m)
    D = np.sort(rng.choice(m // 2, (m, 4)), axis=1)
    keep = np.ones(D.shape, dtype=bool)
    keep[:, 1:] = D[:, 1:] != D[:, :-1]
    keep[rng.integers(0, m, 5000)] = False  # (empty rows)
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(keep.sum(1), out=rp[1:])
    A = _as(CSR(m, m // 2, rp, D[keep].astype(np.int32), rng.standard_normal(int(rp[-1]))), semiring)
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    compare_full(sp.lower(dA, semiring), oracle.lower(A, semiring), semiring, "lower")
    compare_full(sp.offdiag(dA, dA, semiring), oracle.offdiag(A, A, semiring), semiring, "offdiag")
