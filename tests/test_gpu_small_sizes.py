"""Sizes where the launches of a small call change: the column sort's groups in LDS
up to 2^16 entries, scans of one launch up to 2^14 values and of two up to 2^11
tiles of 2^12, the workspace block; narrow and wide column ids, a hub column; against
the oracle, structure and counts exactly."""
import numpy as np
import pytest

import oracle
import paper_2608_09713_amd as sp
from paper_2608_09713_amd.workloads import CSR
from tests.parity import compare_full

pytestmark = pytest.mark.gpu

VDT = {"f64": np.float64, "count": None}


def _matrix(rng, m, n, nnz, hub):
    """nnz distinct entries; the first hub rows hold column 1"""
    key = np.unique(rng.integers(0, m, 2 * nnz) * n + rng.integers(2, n, 2 * nnz))
    key = np.concatenate([np.arange(hub) * n + 1, rng.permutation(key)[:nnz - hub]])
    key.sort()
    assert len(key) == nnz
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=m), out=rp[1:])
    return CSR(m, n, rp, (key % n).astype(np.int32), rng.standard_normal(nnz))


@pytest.mark.parametrize("m,n,nnz,hub", [
    (1, 3, 1, 1),
    (4095, 4097, 4000, 0),
    (1 << 14, 1 << 20, (1 << 14) + 1, 2500),         # a group for the second launch, in LDS
    ((1 << 14) - 1, 5000, (1 << 16) - 1, 300),       # the row scan's last one-launch size
    (1 << 14, 1 << 26, 1 << 16, 5000),               # the last sort of few entries; a group past the LDS
    ((1 << 14) + 1, 1 << 26, (1 << 16) + 1, 5),      # past both
    ((1 << 23) + 3, 1 << 20, 60000, 2),              # 2049 tiles of row counts: three launches
    ((1 << 23) - 1, 1 << 20, 60000, 2),              # 2048: two
])
@pytest.mark.parametrize("semiring", ["f64", "count"])
def test_small_sizes(m, n, nnz, hub, semiring):
    A = _matrix(np.random.default_rng(nnz + m), m, n, nnz, hub)
    A = A.with_values(None if VDT[semiring] is None else A.values.astype(VDT[semiring]))
    print(f"[small sizes {semiring}] m={m} n={n} nnz={A.nnz} hub={hub}", flush=True)
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    ref = oracle.lower(A, semiring)
    compare_full(sp.lower(dA, semiring), ref, semiring, "lower")
    if m < 20000 and hub < 1000:
        compare_full(sp.offdiag(dA, dA, semiring), oracle.offdiag(A, A, semiring), semiring, "offdiag")


@pytest.mark.parametrize("m,n,nnz,lo,width", [
    (1 << 14, 1 << 20, 60000, 5000, 4096),       # one group of high bits, past the LDS: full passes instead
    (1 << 14, 1 << 20, 4097, 8192, 4096),        # just past it
    (1 << 14, 1 << 20, 4096, 8192, 4096),        # and just within
    (1 << 12, 1 << 26, 1 << 16, 70000, 4096),    # columns too wide for few entries' groups
    (1 << 12, (1 << 31) - 1, 1000, (1 << 31) - 2000, 1900),
    (300, (1 << 20) + 1, 2000, 0, (1 << 20) + 1),  # 21 bits
])
@pytest.mark.parametrize("semiring", ["f64", "count"])
def test_few_entries_crowded_or_wide(m, n, nnz, lo, width, semiring):
    """Few entries that the sort in groups does not suit; one-shot, planned (the
    matrices have fewer entries than columns) and off the diagonal."""
    rng = np.random.default_rng(nnz + width)
    key = np.unique(rng.integers(0, m, 3 * nnz) * np.int64(n) + lo + rng.integers(0, width, 3 * nnz))
    key = np.sort(rng.permutation(key)[:nnz])
    assert len(key) == nnz
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=m), out=rp[1:])
    A = CSR(m, n, rp, (key % n).astype(np.int32), rng.standard_normal(nnz))
    A = A.with_values(None if VDT[semiring] is None else A.values)
    print(f"[few entries {semiring}] m={m} n={n} nnz={nnz} width={width}", flush=True)
    dA = sp.DeviceCSR.from_host(A, "cuda:0")
    ref = oracle.lower(A, semiring)
    compare_full(sp.lower(dA, semiring), ref, semiring, "lower")
    plan, C = sp.lower_plan(dA, semiring)
    compare_full(C, ref, semiring, "plan")
    B = A if VDT[semiring] is None else A.with_values(A.values * 2 + 1)
    got = plan.execute(None if VDT[semiring] is None else sp.DeviceCSR.from_host(B, "cuda:0").values)
    compare_full(got, oracle.lower(B, semiring), semiring, "execute")
    plan.close()
    if n < 1 << 28:  # (dense column starts)
        compare_full(sp.offdiag(dA, dA, semiring), oracle.offdiag(A, A, semiring), semiring, "offdiag")
