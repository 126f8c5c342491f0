"""The mirror's column slabs: tiles of few long rows and of many short or empty
ones, keys of one to four digit passes, slabs of equal width at and past
the number counted by row searches; against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2608_09713_amd as sp
from tests.parity import compare_full

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    return torch.device("cuda:0")


def _raw(dev, rp, ci, n, vals=None):
    import torch
    up = lambda x: torch.from_numpy(x).to(dev)
    return sp.DeviceCSR(len(rp) - 1, n, up(rp), up(ci), None if vals is None else up(vals), len(ci))


def _lower(rng, m, lens):
    """lower-triangular rows of about the given lengths (at most row + 1)"""
    rows = np.flatnonzero(lens)
    cols = [np.sort(rng.choice(i + 1, size=min(i + 1, int(lens[i])), replace=False)) if 8 * lens[i] > i
            else np.unique(rng.integers(0, i + 1, int(lens[i]))) for i in rows]
    n = np.zeros(m, dtype=np.int64)
    n[rows] = [len(c) for c in cols]
    rp = np.zeros(m + 1, dtype=np.int64)
    rp[1:] = np.cumsum(n)
    ci = np.concatenate(cols).astype(np.int32)
    return rp, ci, rng.standard_normal(len(ci))


@pytest.mark.parametrize("shape,m,bits", [
    ("long", 4100, 7),     # 33 slabs, rows longer than a tile of records and tiles of few rows
    ("long", 4100, 13),    # one slab, two passes
    ("short", 8192, 7),    # 64 slabs: the most counted by row searches
    ("short", 8193, 7),    # 65: counted by column
    ("short", 9000, 8),    # one pass, more rows per tile than offsets held at once
    ("short", 66000, 0),   # 17-bit keys: three passes, the keys written out
    ("empty", 70000, 0),   # stretches of empty rows longer than any window
    ("empty", 20000, 16),
    ("sparse", (1 << 24) + 70, 0),  # 25-bit keys: four passes
])
def test_mirror_slab_shapes(dev, shape, m, bits, monkeypatch):
    monkeypatch.setenv("SPSYRK_MIRROR_NARROW", str(bits))
    rng = np.random.default_rng(m + bits)
    if shape == "long":
        lens = np.where(np.arange(m) % 97 == 5, m, 3)
    elif shape == "short":
        lens = rng.integers(0, 3, size=m)
    elif shape == "sparse":
        lens = np.zeros(m, dtype=np.int64)
        lens[rng.choice(m, 2000, replace=False)] = 50
        lens[m - 1] = 4000
    else:
        lens = np.where(np.arange(m) % 5000 < 40, 60, 0)
    rp, ci, v = _lower(rng, m, lens)
    print(f"[mirror slab shapes] {shape} m={m} bits={bits} nnz={len(ci)}", flush=True)
    ref = oracle.mirror(m, rp, ci, v)
    compare_full(sp.mirror(_raw(dev, rp, ci, m, v), "f64"), ref, "f64", "mirror f64")
    v32 = v.astype(np.float32)
    ref32 = oracle.mirror(m, rp, ci, v32)
    compare_full(sp.mirror(_raw(dev, rp, ci, m, v32), "f32"), ref32, "f32", "mirror f32")
    M = sp.mirror(_raw(dev, rp, ci, m, None), "count")
    np.testing.assert_array_equal(M.to_host()[0], ref.row_ptr)
    np.testing.assert_array_equal(M.to_host()[1], ref.col_idx)


@pytest.mark.parametrize("m,lens,diagonal", [
    (1 << 20, [3] * 40, False),              # tiles of more rows than are walked, almost all empty
    ((1 << 22) + 5, [2] * 900 + [5000, 3000], False),  # and long rows among them
    (1 << 21, [2] * 30, True),               # the lower part full of diagonals, its records few
    (1 << 15, [1] * 20, False),              # just within the rows that are walked
    ((1 << 15) + 2, [1] * 20, False),
])
def test_mirror_of_mostly_empty_rows(dev, m, lens, diagonal):
    rng = np.random.default_rng(m + len(lens))
    at = np.sort(rng.choice(m - 1, len(lens), replace=False)) + 1
    at[0], at[-1] = 1, m - 1
    rows = np.repeat(at, lens)
    cols = (rng.random(len(rows)) * rows).astype(np.int64)
    key = rows * m + cols
    if diagonal:
        key = np.concatenate([key, np.arange(m) * (m + 1)])
    key = np.unique(key)
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // m, minlength=m), out=rp[1:])
    ci, v = (key % m).astype(np.int32), rng.standard_normal(len(key))
    print(f"[mirror mostly empty] m={m} nnz={len(ci)}", flush=True)
    compare_full(sp.mirror(_raw(dev, rp, ci, m, v), "f64"), oracle.mirror(m, rp, ci, v), "f64", "mirror f64")
    v32 = v.astype(np.float32)
    compare_full(sp.mirror(_raw(dev, rp, ci, m, v32), "f32"), oracle.mirror(m, rp, ci, v32), "f32", "mirror f32")
