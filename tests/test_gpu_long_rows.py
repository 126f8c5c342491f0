"""Heavy rows of more than 512 entries, against the oracle: they go through their
entries two per thread at a time, keep the row at every entry's next position
from window to window (2^17 columns, 2^18 in the symbolic pass) and list the
entries with a stretch in the window for the value tiles."""
import numpy as np
import pytest

import oracle
import paper_2608_09713_amd as sp
from paper_2608_09713_amd.workloads import CSR
from tests.parity import compare_rows

pytestmark = pytest.mark.gpu

VDT = {"f64": np.float64, "f32": np.float32, "count": None, "jaccard": None}
LENS = [513, 1023, 1024, 1025, 1537, 3000]


def _matrix(seed, m, dense):
    """LENS rows near the end and one in the middle, each on columns of its own.
    A column holds 1 to 12 earlier rows, spread evenly, crowded around a window
    edge (so that 0 to 5 and more lie before it) or, with dense, many columns
    hold the rows before one place, so that a window takes several value tiles."""
    rng = np.random.default_rng(seed)
    rows, cols, c = [], [], 0
    for k, ln in enumerate(LENS + [2000]):
        r = m // 2 if k == len(LENS) else m - 1 - 3 * k
        for q in range(ln):
            n = int(rng.integers(1, 13))
            if q % 3 == 0:
                edge = (1 << 17) * int(rng.integers(1, max(2, r >> 17)))
                part = edge + rng.choice(np.arange(-6, 7), n, replace=False)
            elif dense and q % 3 == 1:
                part = rng.integers(0, 40) + 30 * rng.choice(1000, 40, replace=False)
            else:
                part = rng.choice(r, n, replace=False)
            part = np.unique(part[(part >= 0) & (part < r)])
            rows += list(part) + [r]
            cols += [c] * (len(part) + 1)
            c += 1
    rows, cols = np.array(rows, dtype=np.int64), np.array(cols, dtype=np.int64)
    key = np.unique(rows * (c + 3) + cols)
    rows, cols = key // (c + 3), key % (c + 3)
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=m), out=rp[1:])
    A = CSR(m, c + 3, rp, cols.astype(np.int32), rng.standard_normal(len(cols)))
    return A, np.flatnonzero(np.diff(rp) > 512)


@pytest.mark.parametrize("semiring", ["f64", "f32", "count", "jaccard"])
@pytest.mark.parametrize("m,dense", [(100000, True), (1 << 17, False), ((1 << 17) + 1, True), (600000, False),
                                     (600000, True)])
def test_long_rows(semiring, m, dense, monkeypatch):
    A, rows = _matrix(m, m, dense)
    A = A.with_values(None if VDT[semiring] is None else A.values.astype(VDT[semiring]))
    assert len(rows) > len(LENS)
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    print(f"[long rows {semiring}] m={m} nnz={A.nnz}", flush=True)
    rows = np.concatenate([np.arange(0, m, m // 50), rows])
    ref = oracle.lower(A, semiring, rows=rows)
    compare_rows(sp.lower(dA, semiring), ref, rows, semiring, "lower")
    plan, C = sp.lower_plan(dA, semiring)
    compare_rows(C, ref, rows, semiring, "plan")
    if VDT[semiring] is None:
        got, B = plan.execute(None), A
    else:
        B = A.with_values((A.values * 2 - 1).astype(VDT[semiring]))
        got = plan.execute(sp.DeviceCSR.from_host(B, "cuda:0").values)
    compare_rows(got, oracle.lower(B, semiring, rows=rows), rows, semiring, "execute")
    plan.close()
    # off the diagonal (no pruning), in one pass and in two
    off = oracle.offdiag(A, A, semiring, rows=rows)
    compare_rows(sp.offdiag(dA, dA, semiring), off, rows, semiring, "offdiag")
    monkeypatch.setenv("SPSYRK_TWO_PASS", "1")
    compare_rows(sp.offdiag(dA, dA, semiring), off, rows, semiring, "offdiag, two passes")
    compare_rows(sp.lower(dA, semiring), ref, rows, semiring, "lower, two passes")


@pytest.mark.parametrize("semiring", ["f64", "count", "jaccard"])
@pytest.mark.parametrize("lens", [(1, 63, 64), (0, 64, 65), (65, 200)])
def test_batches_of_short_and_long_stretches(semiring, lens):
    """Stretches up to 64 products, which wavefronts walk by themselves where a
    batch of 512 has no longer one, beside batches that do: the first 512
    entries of every row hold the short ones only, the rest all of them; two
    windows in the symbolic pass, three in the numeric one."""
    rng = np.random.default_rng(lens[0])
    m, rows, cols, c = (1 << 18) + 500, [], [], 0
    for k, ln in enumerate([600, 1024, 1500]):
        r = m - 1 - 2 * k
        for q in range(ln):
            n = int(rng.choice([x for x in lens if x <= 64] or lens)) if q < 512 else int(rng.choice(lens))
            # all before one window's end, so that the stretch is not cut
            part = (int(rng.integers(0, 2)) << 17) + rng.choice(1 << 16, n, replace=False)
            rows += list(part) + [r]
            cols += [c] * (n + 1)
            c += 1
    rows, cols = np.array(rows, dtype=np.int64), np.array(cols, dtype=np.int64)
    key = np.unique(rows * c + cols)
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // c, minlength=m), out=rp[1:])
    A = CSR(m, c, rp, (key % c).astype(np.int32), rng.standard_normal(len(key)))
    A = A.with_values(None if VDT[semiring] is None else A.values)
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    print(f"[stretches {lens} {semiring}] nnz={A.nnz}", flush=True)
    rows = np.concatenate([np.arange(0, m, m // 50), [m - 5, m - 3, m - 1]])
    C = sp.lower(dA, semiring)
    assert sp.stats()["heavy_rows"] >= 3 and sp.stats()["cell_rows"] == 0
    compare_rows(C, oracle.lower(A, semiring, rows=rows), rows, semiring, "lower")
    compare_rows(sp.offdiag(dA, dA, semiring), oracle.offdiag(A, A, semiring, rows=rows), rows, semiring, "offdiag")
